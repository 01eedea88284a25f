"""Helpers of the GPU parity tests: move a synthetic round to the device, call
the library through its binding, and compare with the oracle."""
import numpy as np

from oracle import hx_oracle as o

REL = 1e-5     # fp32 costs against the fp64 oracle


def dev(x):
    import torch
    if x is None:
        return None
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def dev_tables(rnd):
    from paper_2605_16637_amd import binding
    calls = binding.to_device(rnd.calls)
    pre = binding.to_device(rnd.pre)
    dec = binding.to_device(rnd.dec)
    links = binding.to_device(rnd.links)
    return calls, pre, dec, links


def fused(ctx, model, calls, pre, dec, links, tail=None, horizon=None, want_ratio=False):
    import torch
    n = int(calls["n"])
    bp = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    bd = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    bc = torch.full((n,), -7.0, dtype=torch.float32, device="cuda:0")
    ratio = torch.full((n,), -7.0, dtype=torch.float32, device="cuda:0") if want_ratio else None
    ctx.hx_score_placements(model, calls, pre, dec, links, tail=tail, horizon=horizon,
                            best_p=bp, best_d=bd, best_cost=bc, ratio=ratio)
    ctx.hx_stream_status()
    out = [bp.cpu().numpy(), bd.cpu().numpy(), bc.cpu().numpy()]
    if want_ratio:
        out.append(ratio.cpu().numpy())
    return out


def assert_costs_close(gpu, ref, what="cost"):
    gpu = np.asarray(gpu, np.float64)
    ref = np.asarray(ref, np.float64)
    assert gpu.shape == ref.shape
    assert np.array_equal(np.isinf(gpu), np.isinf(ref)), f"{what}: infeasible pattern differs"
    assert not np.isnan(gpu).any(), f"{what}: NaN"
    fin = np.isfinite(ref)
    err = np.abs(gpu[fin] - ref[fin]) / np.maximum(np.abs(ref[fin]), 1e-30)
    assert err.size == 0 or err.max() <= REL, f"{what}: max relative error {err.max():.3e}"
    return float(err.max()) if err.size else 0.0


def assert_search_matches(rnd_model, L_in, L_out, pre, dec, links, ores, gp, gd, gc, rows=None):
    """Selected indices equal the oracle's, except where the oracle's cost of
    the GPU's pair is within REL of the oracle's best (a near-tie in fp32);
    best costs within REL; 'no feasible pair' agrees exactly.  `rows` maps the
    compared entries to call indices when only a sample is checked."""
    rows = np.arange(len(gp)) if rows is None else rows
    assert_costs_close(gc, ores.best_cost, "best_cost")
    none_o = ores.best_p < 0
    assert np.array_equal(gp < 0, none_o) and np.array_equal(gd < 0, none_o)
    diff = np.nonzero((gp != ores.best_p) | (gd != ores.best_d))[0]
    for i in diff:
        c = rows[i]
        alt = o.score_one(rnd_model, L_in[c], L_out[c], gp[i], gd[i], pre, dec, links)
        assert np.isfinite(alt) and alt <= ores.best_cost[i] * (1 + REL), \
            f"call {c}: GPU chose ({gp[i]},{gd[i]}) cost {alt}, oracle ({ores.best_p[i]},{ores.best_d[i]}) cost {ores.best_cost[i]}"
    return len(diff)


def many_small_workflows(n_wf, size, large, stride):
    """Row and workflow bounds and successors of n_wf workflows of `size` nodes, but of `large` one in each odd run of `stride` workflows, at another place in each; a node's successors are the next two of its workflow."""
    sizes = np.full(n_wf, size, np.int64)
    runs = np.arange(1, n_wf // stride, 2)
    sizes[runs * stride + runs * 7 % stride] = large
    wf_ptr = np.concatenate([[0], np.cumsum(sizes)])
    v, end = np.arange(wf_ptr[-1]), np.repeat(wf_ptr[1:], sizes)
    there = v[:, None] + np.array([1, 2]) < end[:, None]
    row_ptr = np.concatenate([[0], np.cumsum(there.sum(1))])
    return row_ptr.astype(np.int32), (v[:, None] + np.array([1, 2]))[there].astype(np.int32), wf_ptr.astype(np.int32)


# (workflows, nodes of each, of the large ones, workflows to an odd run): many workflows a wavefront and several runs a workgroup, some of
# which have a workflow that no wavefront can take; runs as long as the workgroups', so that each of their numbers is met
FALLBACKS = [(18432, 4, 65, 36), (18432, 4, 65, 72), (40000, 2, 65, 76), (40000, 2, 200, 300), (70000, 1, 65, 128), (70000, 1, 65, 256),
             (20000, 0, 65, 128), (1000, 30, 65, 4), (300, 9, 70, 4)]
