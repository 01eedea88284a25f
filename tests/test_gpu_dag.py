"""GPU parity of the horizon path (standalone node cost, critical path in its
single-pass and level-synchronous forms, incremental append) and of the
commit step, against the CPU oracle, through the C ABI."""
import numpy as np
import pytest

from oracle import hx_oracle as o
from paper_2605_16637_amd import synth
from gpu_helpers import FALLBACKS, assert_costs_close, dev, many_small_workflows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2605_16637_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


def gpu_cp(ctx, row_ptr, col, cost32, wf_ptr, max_sweeps=0, check=True):
    import torch
    n, n_wf = len(row_ptr) - 1, len(wf_ptr) - 1
    rem = torch.full((n,), -1.0, device="cuda:0"); tail = torch.full((n,), -1.0, device="cuda:0")
    level = torch.full((n,), -1, dtype=torch.int32, device="cuda:0")
    hor = torch.full((n_wf,), -1.0, device="cuda:0")
    ctx.hx_critical_path(dev(np.asarray(row_ptr, np.int32)), dev(np.asarray(col, np.int32)), dev(cost32),
                         dev(np.asarray(wf_ptr, np.int32)), rem, tail, level, hor, max_sweeps=max_sweeps)
    if check:
        ctx.hx_stream_status()
    return rem.cpu().numpy(), tail.cpu().numpy(), level.cpu().numpy(), hor.cpu().numpy()


def assert_cp_bit_exact(got, want):
    rem, tail, level, hor = got
    orem, otail, olevel, ohor = want          # fp64 holders of exact fp32 values
    assert np.array_equal(level, olevel)
    assert np.array_equal(rem, orem.astype(np.float32)) and np.array_equal(rem.astype(np.float64), orem)
    assert np.array_equal(tail.astype(np.float64), otail)
    assert np.array_equal(hor.astype(np.float64), ohor)


@pytest.mark.parametrize("name,seed", [("tiny", 1), ("mid", 1), ("mid", 2)])
def test_node_cost_and_critical_path(ctx, name, seed):
    import torch
    from paper_2605_16637_amd import binding
    rnd = synth.make_round(name, seed)
    d = rnd.dag
    ocost = o.node_cost(rnd.model, d.L_in, d.L_out, rnd.types, rnd.links)
    gcost = torch.empty(d.n_nodes, device="cuda:0")
    ctx.hx_node_cost(rnd.model, dev(d.L_in), dev(d.L_out), dev(rnd.types["flops"]), dev(rnd.types["hbm_bw"]),
                     binding.to_device(rnd.links), gcost)
    ctx.hx_stream_status()
    assert_costs_close(gcost.cpu().numpy(), ocost, "node cost")
    # the pass itself: same fp32 costs into both sides -> identical bits
    cost32 = ocost.astype(np.float32)
    want = o.critical_path(d.succ_row_ptr, d.succ_col, cost32.astype(np.float64), d.wf_ptr, round_f32=True)
    got = gpu_cp(ctx, d.succ_row_ptr, d.succ_col, cost32, d.wf_ptr)
    assert_cp_bit_exact(got, want)
    got = gpu_cp(ctx, d.succ_row_ptr, d.succ_col, cost32, d.wf_ptr, max_sweeps=int(want[2].max()) + 2)
    assert_cp_bit_exact(got, want)
    # and against the fp64 definition, within the fp32 tolerance
    want64 = o.critical_path(d.succ_row_ptr, d.succ_col, ocost, d.wf_ptr, round_f32=False)
    assert_costs_close(got[0], want64[0], "rem"); assert_costs_close(got[3], want64[3], "horizon")
    # whole chain on the GPU: its own node cost into its own pass
    got2 = gpu_cp(ctx, d.succ_row_ptr, d.succ_col, gcost.cpu().numpy(), d.wf_ptr)
    assert np.array_equal(got2[2], want[2])
    assert_costs_close(got2[0], want64[0], "rem, GPU cost"); assert_costs_close(got2[3], want64[3], "horizon, GPU cost")


@pytest.mark.parametrize("T", [1, 3, 4, 5, 8])
def test_node_cost_of_many_nodes(ctx, T):
    # From 393216 nodes on (256 compute units; 786432 if there are more than four classes) a thread takes four; beyond 2097152 it comes
    # back for more; more than four classes are taken all at once up to 65536 or 131072 nodes.  Any part of the array on its own,
    # short enough for a node a thread, has the same bits, and nothing is written past the end.
    import torch
    from paper_2605_16637_amd import binding
    rng = np.random.default_rng(T)
    types = dict(flops=rng.uniform(1e14, 3e15, T).astype(np.float32), hbm_bw=rng.uniform(1e12, 8e12, T).astype(np.float32))
    links = dict(n_types=T, bw=rng.uniform(1e10, 1e11, T * T).astype(np.float32),
                 latency=rng.uniform(0, 0.01, T * T).astype(np.float32) if T % 2 else None)
    most = 2097152 + 1025
    L, O = rng.integers(0, 32769, most).astype(np.int32), rng.integers(0, 4097, most).astype(np.int32)
    dL, dO, tF, tB, dl = dev(L), dev(O), dev(types["flops"]), dev(types["hbm_bw"]), binding.to_device(links)

    def cost(i, n):
        out = torch.full((n + 64,), -7.0, device="cuda:0")
        ctx.hx_node_cost(synth.MODEL, dL[i:i + n], dO[i:i + n], tF, tB, dl, out[:n])
        ctx.hx_stream_status()
        assert bool((out[n:] == -7.0).all())
        return out[:n].cpu().numpy()

    parts = np.concatenate([cost(i, min(200000, most - i)) for i in range(0, most, 200000)])
    for n in (1, 65536, 65537, 131072, 131073, 262144, 262145, 393215, 393217, 524287, 786431, 786433, most):
        assert np.array_equal(cost(0, n), parts[:n])
    some = rng.choice(most, 2000, replace=False)
    assert_costs_close(parts[some], o.node_cost(synth.MODEL, L[some], O[some], types, links), "node cost")


def test_critical_path_stress_full_size(ctx):
    # 100 000 workflows, 2.0 M nodes, ~3.4 M edges, depth up to 32
    rnd = synth.make_round("cp", 1)
    d = rnd.dag
    assert d.n_wf == 100000 and 1.9e6 < d.n_nodes < 2.1e6
    rng = np.random.default_rng(3)
    cost32 = o.node_cost(rnd.model, d.L_in, d.L_out, rnd.types, rnd.links).astype(np.float32)
    want = o.critical_path(d.succ_row_ptr, d.succ_col, cost32.astype(np.float64), d.wf_ptr, round_f32=True)
    assert 24 <= want[2].max() <= 31
    got = gpu_cp(ctx, d.succ_row_ptr, d.succ_col, cost32, d.wf_ptr)
    assert_cp_bit_exact(got, want)
    got = gpu_cp(ctx, d.succ_row_ptr, d.succ_col, cost32, d.wf_ptr, max_sweeps=int(want[2].max()) + 2)
    assert_cp_bit_exact(got, want)


def test_single_pass_edge_cases(ctx):
    # empty graph, workflows without nodes, one huge workflow (walked outside LDS),
    # more workflows than one block takes
    got = gpu_cp(ctx, [0], [], np.zeros(0, np.float32), [0])
    assert all(x.size == 0 for x in got)
    got = gpu_cp(ctx, [0, 0], [], np.array([2.5], np.float32), [0, 0, 1, 1])
    assert list(got[3]) == [0.0, 2.5, 0.0] and got[0][0] == 2.5 and got[2][0] == 0
    n = 20000                                  # chain longer than the LDS slice
    rng = np.random.default_rng(4)
    cost32 = rng.uniform(0.1, 2.0, n).astype(np.float32)
    row_ptr = np.minimum(np.arange(n + 1), n - 1).astype(np.int32)
    col = np.arange(1, n, dtype=np.int32)
    want = o.critical_path(row_ptr, col, cost32.astype(np.float64), [0, n], round_f32=True)
    assert_cp_bit_exact(gpu_cp(ctx, row_ptr, col, cost32, [0, n]), want)
    assert want[2][0] == n - 1
    dag = synth.gen_dag(rng, 1000, 1, 3, 2, 3)  # 1000 tiny workflows, some of one node
    c32 = rng.uniform(0.1, 2.0, dag.n_nodes).astype(np.float32)
    want = o.critical_path(dag.succ_row_ptr, dag.succ_col, c32.astype(np.float64), dag.wf_ptr, round_f32=True)
    assert_cp_bit_exact(gpu_cp(ctx, dag.succ_row_ptr, dag.succ_col, c32, dag.wf_ptr), want)


def test_sweeps_accept_any_numbering_and_report_cycles(ctx):
    from paper_2605_16637_amd import binding
    rnd = synth.make_round("mid", 4)
    d = rnd.dag
    rng = np.random.default_rng(5)
    cost32 = rng.uniform(0.5, 3.0, d.n_nodes).astype(np.float32)
    perm = rng.permutation(d.n_nodes)
    inv = np.argsort(perm)
    deg = np.diff(d.succ_row_ptr)[inv]
    rp = np.zeros(d.n_nodes + 1, np.int32); rp[1:] = np.cumsum(deg)
    src_old = np.repeat(inv, deg)
    offs = np.arange(int(deg.sum())) - np.repeat(rp[:-1], deg)
    col = perm[d.succ_col[d.succ_row_ptr[src_old] + offs]].astype(np.int32)
    want = o.critical_path(rp, col, cost32[inv].astype(np.float64), [0, d.n_nodes], round_f32=True)
    got = gpu_cp(ctx, rp, col, cost32[inv], [0, d.n_nodes], max_sweeps=int(want[2].max()) + 2)
    assert_cp_bit_exact(got, want)
    # the single pass refuses this numbering instead of returning wrong values silently
    gpu_cp(ctx, rp, col, cost32[inv], [0, d.n_nodes], check=False)
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -3
    # a cycle: no fixed point within the limit
    gpu_cp(ctx, [0, 1, 2, 3], [1, 2, 0], np.ones(3, np.float32), [0, 3], max_sweeps=8, check=False)
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -3
    # too few sweeps for the depth is reported the same way
    gpu_cp(ctx, d.succ_row_ptr, d.succ_col, cost32, d.wf_ptr, max_sweeps=2, check=False)
    with pytest.raises(binding.HxError):
        ctx.hx_stream_status()


@pytest.mark.parametrize("edge,code", [((1, 4), -3),     # into a later workflow that shares the block
                                       ((4, 1), -3),     # backwards, into an earlier workflow
                                       ((2, 2), -3),     # onto itself
                                       ((1, 9), -3),     # past the last node
                                       (None, 0)])
def test_single_pass_reports_edges_that_leave_their_workflow(ctx, edge, code):
    from paper_2605_16637_amd import binding
    # two chains of three nodes, 0-1-2 and 3-4-5, plus one extra edge
    succ = {0: [1], 1: [2], 2: [], 3: [4], 4: [5], 5: []}
    if edge:
        succ[edge[0]] = succ[edge[0]] + [edge[1]]
    row_ptr = np.cumsum([0] + [len(succ[v]) for v in range(6)]).astype(np.int32)
    col = np.array([u for v in range(6) for u in succ[v]], np.int32)
    cost32 = np.arange(1, 7, dtype=np.float32)
    got = gpu_cp(ctx, row_ptr, col, cost32, [0, 3, 6], check=False)
    if code == 0:
        ctx.hx_stream_status()
        assert list(got[0]) == [6.0, 5.0, 3.0, 15.0, 11.0, 6.0] and list(got[3]) == [6.0, 15.0]
        assert list(got[2]) == [2, 1, 0, 2, 1, 0]
    else:
        with pytest.raises(binding.HxError) as e:
            ctx.hx_stream_status()
        assert e.value.code == code
        # the workflow the bad edge does not start in is untouched by it
        other = slice(3, 6) if edge[0] < 3 else slice(0, 3)
        assert list(got[0][other]) == ([15.0, 11.0, 6.0] if edge[0] < 3 else [6.0, 5.0, 3.0])


def _random_forest(rng, sizes, fan_out, p_second=0.5):
    """Workflows of the given sizes, ids parent-first and workflow-contiguous; every node but a workflow's
    first draws one parent (and sometimes a second) among the earlier nodes of its workflow that still
    have fewer than `fan_out` successors."""
    succ, wf_ptr = [], [0]
    for size in sizes:
        base = len(succ)
        succ.extend([] for _ in range(size))
        for i in range(1, size):
            free = [u for u in range(base, base + i) if len(succ[u]) < fan_out]
            for u in set(rng.choice(free, size=min(len(free), 1 + (rng.random() < p_second)), replace=False).tolist()):
                succ[u].append(base + i)
        wf_ptr.append(len(succ))
    row_ptr = np.cumsum([0] + [len(x) for x in succ]).astype(np.int32)
    col = np.array([u for x in succ for u in sorted(x)], np.int32)
    return row_ptr, col, np.array(wf_ptr, np.int32)


@pytest.mark.parametrize("sizes,fan_out,seed", [
    ([40] * 30, 12, 1),                         # nodes with up to 12 successors
    ([3, 900, 5, 700, 1, 650, 20] * 3, 4, 2),   # neighbours that do not fit one block's LDS together
    ([60, 1390, 2, 1400, 1401, 7, 1399], 9, 3), # at and around the most one block stages; wide nodes too
    ([1] * 300 + [2500] + [4] * 100, 3, 4),     # one workflow too large for LDS between small ones
])
def test_single_pass_wide_nodes_and_runs_of_workflows(ctx, sizes, fan_out, seed):
    rng = np.random.default_rng(seed)
    row_ptr, col, wf_ptr = _random_forest(rng, sizes, fan_out)
    assert (np.diff(row_ptr).max() > 4) == (fan_out > 4)
    cost32 = rng.uniform(0.1, 2.0, len(row_ptr) - 1).astype(np.float32)
    want = o.critical_path(row_ptr, col, cost32.astype(np.float64), wf_ptr, round_f32=True)
    assert_cp_bit_exact(gpu_cp(ctx, row_ptr, col, cost32, wf_ptr), want)
    # a wide node with one edge out of its workflow is reported
    wide = int(np.argmax(np.diff(row_ptr)))
    if row_ptr[wide + 1] - row_ptr[wide] > 4 and wf_ptr[1] <= wide:
        col2 = col.copy(); col2[row_ptr[wide + 1] - 1] = 0
        gpu_cp(ctx, row_ptr, col2, cost32, wf_ptr, check=False)
        from paper_2605_16637_amd import binding
        with pytest.raises(binding.HxError) as e:
            ctx.hx_stream_status()
        assert e.value.code == -3


def gpu_horizons(ctx, rnd, row_ptr, col, L_in, L_out, wf_ptr, check=True):
    import torch
    from paper_2605_16637_amd import binding
    n, n_wf = len(row_ptr) - 1, len(wf_ptr) - 1
    f = lambda v: torch.full((n,), v, device="cuda:0")
    cost, rem, tail = f(-1.0), f(-1.0), f(-1.0)
    level = torch.full((n,), -1, dtype=torch.int32, device="cuda:0")
    hor = torch.full((n_wf,), -1.0, device="cuda:0")
    ctx.hx_horizons(rnd.model, dev(np.asarray(row_ptr, np.int32)), dev(np.asarray(col, np.int32)),
                    dev(np.asarray(L_in, np.int32)), dev(np.asarray(L_out, np.int32)),
                    dev(rnd.types["flops"]), dev(rnd.types["hbm_bw"]), binding.to_device(rnd.links),
                    dev(np.asarray(wf_ptr, np.int32)), cost, rem, tail, level, hor)
    if check:
        ctx.hx_stream_status()
    return cost.cpu().numpy(), (rem.cpu().numpy(), tail.cpu().numpy(), level.cpu().numpy(), hor.cpu().numpy())


@pytest.mark.parametrize("name,seed", [("tiny", 1), ("mid", 3), ("large", 1), ("cp", 2)])
def test_horizons_in_one_launch(ctx, name, seed):
    """Node cost and critical path in one launch: the cost within tolerance of the oracle's and bit for
    bit what hx_node_cost gives; the pass bit for bit the oracle's fp32 pass on those costs."""
    import torch
    from paper_2605_16637_amd import binding
    rnd = synth.make_round(name, seed)
    d = rnd.dag
    gcost, got = gpu_horizons(ctx, rnd, d.succ_row_ptr, d.succ_col, d.L_in, d.L_out, d.wf_ptr)
    assert_costs_close(gcost, o.node_cost(rnd.model, d.L_in, d.L_out, rnd.types, rnd.links), "node cost")
    two = torch.empty(d.n_nodes, device="cuda:0")
    ctx.hx_node_cost(rnd.model, dev(d.L_in), dev(d.L_out), dev(rnd.types["flops"]), dev(rnd.types["hbm_bw"]),
                     binding.to_device(rnd.links), two)
    assert np.array_equal(gcost, two.cpu().numpy())
    want = o.critical_path(d.succ_row_ptr, d.succ_col, gcost.astype(np.float64), d.wf_ptr, round_f32=True)
    assert_cp_bit_exact(got, want)


@pytest.mark.parametrize("sizes,fan_out,seed", [
    ([40] * 30, 12, 1), ([3, 900, 5, 700, 1, 650, 20] * 3, 4, 2), ([1] * 300 + [2500] + [4] * 100, 3, 4), ([], 3, 5), ([0, 1, 0], 3, 6)])
def test_horizons_in_one_launch_wide_nodes_and_runs(ctx, sizes, fan_out, seed):
    rng = np.random.default_rng(seed)
    rnd = synth.make_round("tiny", 1)
    row_ptr, col, wf_ptr = _random_forest(rng, sizes, fan_out)
    n = len(row_ptr) - 1
    L_in, L_out = rng.integers(64, 8000, n).astype(np.int32), rng.integers(16, 2000, n).astype(np.int32)
    gcost, got = gpu_horizons(ctx, rnd, row_ptr, col, L_in, L_out, wf_ptr)
    if n == 0:
        assert all(x.size == 0 for x in got[:3]) and list(got[3]) == [0.0] * (len(wf_ptr) - 1)
        return
    assert_costs_close(gcost, o.node_cost(rnd.model, L_in, L_out, rnd.types, rnd.links), "node cost")
    want = o.critical_path(row_ptr, col, gcost.astype(np.float64), wf_ptr, round_f32=True)
    assert_cp_bit_exact(got, want)


@pytest.mark.parametrize("sizes,fan_out,seed", [
    ([64] * 5 + [1] * 40, 3, 1), ([63, 64, 1, 64, 2, 62] * 60, 2, 2),     # a wavefront's lanes, just filled
    ([65] + [3] * 40, 3, 3),                                               # one workflow too large for them
    ([0, 0, 64, 0, 1, 0] * 9, 3, 4), ([2, 1], 2, 5), ([4], 3, 6),          # empty ones; fewer edges than one load takes
    ([30] * 40 + [2], 9, 7), ([40] * 20, 30, 8), ([64] * 12, 63, 9),       # successors beyond four: in LDS, more than there is room for
    ([8] * 9000, 3, 10), ([20] * 5000, 3, 11)])                            # several workflows a wavefront
def test_small_workflows_by_wavefronts(ctx, sizes, fan_out, seed):
    """Wavefronts of whole workflows: in one launch with the node cost, and in the sweeps (nodes renumbered backwards)."""
    rng = np.random.default_rng(seed)
    rnd = synth.make_round("tiny", 1)
    row_ptr, col, wf_ptr = _random_forest(rng, sizes, fan_out)
    n = len(row_ptr) - 1
    L_in, L_out = rng.integers(64, 8000, n).astype(np.int32), rng.integers(16, 2000, n).astype(np.int32)
    gcost, got = gpu_horizons(ctx, rnd, row_ptr, col, L_in, L_out, wf_ptr)
    want = o.critical_path(row_ptr, col, gcost.astype(np.float64), wf_ptr, round_f32=True)
    assert_cp_bit_exact(got, want)
    # node v of a workflow [s, e) becomes s + e - 1 - v
    wf = np.repeat(np.arange(len(sizes)), sizes)
    to = wf_ptr[wf] + wf_ptr[wf + 1] - 1 - np.arange(n)
    src = np.repeat(np.arange(n), np.diff(row_ptr))
    order = np.lexsort((to[col], to[src]))
    back_ptr = np.concatenate([[0], np.cumsum(np.bincount(to[src], minlength=n))]).astype(np.int32)
    cost = np.empty_like(gcost)
    cost[to] = gcost
    back = gpu_cp(ctx, back_ptr, to[col][order].astype(np.int32), cost, wf_ptr, max_sweeps=80)
    for x, y in zip(back[:3], got[:3]):
        assert np.array_equal(x[to], y)
    assert np.array_equal(back[3], got[3])


@pytest.mark.parametrize("graph", FALLBACKS)
def test_workgroups_with_a_workflow_too_large_for_a_wavefront(ctx, graph):
    """Many small workflows, some of a workgroup's too large for its wavefronts: every workflow of that workgroup is walked all the same."""
    rng = np.random.default_rng(graph[0])
    rnd = synth.make_round("tiny", 1)
    row_ptr, col, wf_ptr = many_small_workflows(*graph)
    n = len(row_ptr) - 1
    L_in, L_out = rng.integers(64, 8000, n).astype(np.int32), rng.integers(16, 2000, n).astype(np.int32)
    gcost, got = gpu_horizons(ctx, rnd, row_ptr, col, L_in, L_out, wf_ptr)
    want = o.critical_path(row_ptr, col, gcost.astype(np.float64), wf_ptr, round_f32=True)
    assert_cp_bit_exact(got, want)
    assert_cp_bit_exact(gpu_cp(ctx, row_ptr, col, gcost, wf_ptr), want)
    assert_cp_bit_exact(gpu_cp(ctx, row_ptr, col, gcost, wf_ptr, max_sweeps=graph[2] + 2), want)
    # one bound that is none: the two workflows beside it get no values, all others theirs, and it is reported
    from paper_2605_16637_amd import binding
    k = graph[3] + 5
    bad = wf_ptr.copy()
    bad[k] = -5
    _, odd = gpu_horizons(ctx, rnd, row_ptr, col, L_in, L_out, bad, check=False)
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -6      # HX_ERR_INDEX
    keep = np.ones(n, bool)
    keep[wf_ptr[k - 1]:wf_ptr[k + 1]] = False
    for x, y in zip(odd[:3], want[:3]):
        assert np.array_equal(x[keep].astype(np.float64), y[keep])
    keep = np.ones(len(wf_ptr) - 1, bool)
    keep[k - 1:k + 1] = False
    assert np.array_equal(odd[3][keep].astype(np.float64), want[3][keep])


def fetch(raw):
    """Copy a borrowed device array of the context to the host (device-to-device copy into a tensor first)."""
    import ctypes
    import torch
    out = torch.empty(raw.numel(), dtype=raw.dtype, device="cuda:0")
    if raw.numel():
        torch.cuda.synchronize()
        hip = ctypes.CDLL("libamdhip64.so")
        rc = hip.hipMemcpy(ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(raw.addr), ctypes.c_size_t(raw.numel() * 4), 3)
        assert rc == 0
    return out.cpu().numpy()


def view(ctx, n, n_wf):
    rem, tail, level, hor, n_nodes = ctx.hx_dag_view(n_wf)
    assert n_nodes == n
    return fetch(rem), fetch(tail), fetch(level), fetch(hor)


@pytest.mark.parametrize("seed,n_live,rounds", [(1, 40, 12), (2, 700, 8)])
def test_incremental_append_equals_full_recompute(ctx, seed, n_live, rounds):
    gen = synth.StreamGen(seed, n_live, final_lo=4, final_hi=14)
    rng = np.random.default_rng(seed)
    ctx.hx_dag_reserve(200000, 300000, 50000, 16)
    prow = np.zeros(1, np.int32); pcol = np.zeros(0, np.int32)
    cost_all = np.zeros(0, np.float32); wf_all = np.zeros(0, np.int32)
    prev_h = np.zeros(0)
    for r in range(rounds):
        b = gen.next_batch()
        cost32 = rng.uniform(0.2, 4.0, b["n_new"]).astype(np.float32)
        ctx.hx_dag_append(dev(b["parent_row_ptr"]), dev(b["parent_col"]), dev(cost32), dev(b["wf"]))
        ctx.hx_stream_status()
        prow = np.concatenate([prow, prow[-1] + b["parent_row_ptr"][1:]]).astype(np.int32)
        pcol = np.concatenate([pcol, b["parent_col"]]); cost_all = np.concatenate([cost_all, cost32])
        wf_all = np.concatenate([wf_all, b["wf"]])
        n_wf = b["n_wf_total"]
        want = o.critical_path_by_parents(prow, pcol, cost_all.astype(np.float64), wf_all, n_wf, round_f32=True)
        got = view(ctx, cost_all.size, n_wf)
        assert np.array_equal(got[2], want[2])
        assert np.array_equal(got[0].astype(np.float64), want[0]) and np.array_equal(got[1].astype(np.float64), want[1])
        assert np.array_equal(got[3].astype(np.float64), want[3])
        assert (want[3][:prev_h.size] >= prev_h).all()      # horizons only grow under reveal
        prev_h = want[3]
    assert want[2].max() >= 3


def test_observed_costs_replace_estimates(ctx):
    """Sec. 5.1: estimates are replaced by observed latencies when they become known.  Costs of existing nodes
    go up and down; rem, tail and horizons must equal a full recomputation, and appending goes on from there."""
    gen = synth.StreamGen(9, 300, final_lo=5, final_hi=25)
    rng = np.random.default_rng(9)
    ctx.hx_dag_reserve(100000, 150000, 20000, 32)
    prow = np.zeros(1, np.int32); pcol = np.zeros(0, np.int32)
    cost_all = np.zeros(0, np.float32); wf_all = np.zeros(0, np.int32)

    def check(n_wf):
        want = o.critical_path_by_parents(prow, pcol, cost_all.astype(np.float64), wf_all, n_wf, round_f32=True)
        got = view(ctx, cost_all.size, n_wf)
        assert np.array_equal(got[2], want[2])
        for k in (0, 1, 3):
            assert np.array_equal(got[k].astype(np.float64), want[k]), k
        return want

    for r in range(8):
        b = gen.next_batch()
        c32 = rng.uniform(0.2, 4.0, b["n_new"]).astype(np.float32)
        ctx.hx_dag_append(dev(b["parent_row_ptr"]), dev(b["parent_col"]), dev(c32), dev(b["wf"]))
        prow = np.concatenate([prow, prow[-1] + b["parent_row_ptr"][1:]]).astype(np.int32)
        pcol = np.concatenate([pcol, b["parent_col"]]); cost_all = np.concatenate([cost_all, c32]); wf_all = np.concatenate([wf_all, b["wf"]])
        n_wf = b["n_wf_total"]
        if r in (3, 5, 7):
            before = check(n_wf)
            ids = rng.choice(cost_all.size, max(1, cost_all.size // 10), replace=False).astype(np.int32)
            new = (cost_all[ids] * rng.choice([0.0, 0.3, 1.0, 2.5], ids.size)).astype(np.float32)     # down, same, up
            ctx.hx_dag_set_cost(dev(ids), dev(new))
            ctx.hx_stream_status()
            cost_all[ids] = new
            after = check(n_wf)
            assert (after[3] < before[3]).any() and (after[3] > before[3]).any()       # horizons moved both ways
    from paper_2605_16637_amd import binding
    ctx.hx_dag_set_cost(dev(np.array([0, 10**7], np.int32)), dev(np.array([1.0, 1.0], np.float32)))
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -6


@pytest.mark.parametrize("reach,most,cross", [(1, 1, 0.0), (3, 2, 0.3), (9, 6, 0.1), (400, 3, 1.0)])
def test_append_of_any_graph(ctx, reach, most, cross):
    """Parents of the same batch (the first parents above a node are followed through them), up to `most` parents,
    also of other workflows, nodes that cost nothing; then other costs for some of them.  Batches of one node to some
    workgroups full."""
    rng = np.random.default_rng(reach)
    ctx.hx_dag_reserve(6000, 40000, 64, 1500)
    prow, pcol = [0], []
    wf = np.zeros(0, np.int32); cost = np.zeros(0, np.float32)

    def check():
        want = o.critical_path_by_parents(np.array(prow, np.int32), np.array(pcol, np.int32), cost.astype(np.float64), wf, 64, round_f32=True)
        got = view(ctx, cost.size, 64)
        assert np.array_equal(got[2], want[2])
        for k in (0, 1, 3):
            assert np.array_equal(got[k].astype(np.float64), want[k]), k

    for n_new in (1, 7, 64, 300, 1, 900):
        n0, e0 = cost.size, len(pcol)
        row = [0]
        for v in range(n0, n0 + n_new):
            k = min(v, int(rng.integers(0 if rng.random() < 0.02 else 1, most + 1)))
            pcol.extend(rng.choice(np.arange(max(0, v - reach), v), min(k, reach, v), replace=False).tolist())
            row.append(len(pcol) - e0)
        prow.extend((e0 + np.array(row[1:])).tolist())
        w = rng.integers(0, 64, n_new).astype(np.int32)
        same = rng.random(n_new) >= cross
        wf = np.concatenate([wf, np.where(same, 5, w).astype(np.int32)])
        c = np.where(rng.random(n_new) < 0.3, 0.0, rng.uniform(0.1, 3.0, n_new)).astype(np.float32)
        cost = np.concatenate([cost, c])
        ctx.hx_dag_append(dev(np.array(row, np.int32)), dev(np.array(pcol[e0:], np.int32)), dev(c), dev(wf[n0:]))
        ctx.hx_stream_status()
        check()
        ids = rng.choice(cost.size, max(1, cost.size // 3), replace=False).astype(np.int32)
        cost[ids] = np.where(rng.random(ids.size) < 0.5, 0.0, rng.uniform(0.1, 3.0, ids.size)).astype(np.float32)
        ctx.hx_dag_set_cost(dev(ids), dev(cost[ids]))
        ctx.hx_stream_status()
        check()


@pytest.mark.parametrize("reach,most", [(1, 1), (3, 2), (9, 6)])
def test_costs_of_minus_zero_are_zeros(ctx, reach, most):
    """A cost of -0.0 is not below 0: whatever is appended under such a node later raises its rem as it does any other's."""
    rng = np.random.default_rng(20 + reach)
    ctx.hx_dag_reserve(700, 4000, 1, 700)
    prow, pcol, cost = [0], [], np.zeros(0, np.float32)
    for n_new in (1, 40, 1, 200, 300):
        n0, e0 = cost.size, len(pcol)
        for v in range(n0, n0 + n_new):
            pcol.extend(rng.choice(np.arange(max(0, v - reach), v), min(v, reach, int(rng.integers(1, most + 1))), replace=False).tolist())
            prow.append(len(pcol))
        c = rng.choice(np.array([-0.0, 0.0, 0.25, 1.5], np.float32), n_new)
        c[0] = -0.0
        cost = np.concatenate([cost, c])
        ctx.hx_dag_append(dev(np.array(prow[n0:], np.int32) - e0), dev(np.array(pcol[e0:], np.int32)), dev(c), dev(np.zeros(n_new, np.int32)))
        ctx.hx_stream_status()
        want = o.critical_path_by_parents(np.array(prow, np.int32), np.array(pcol, np.int32), cost.astype(np.float64), np.zeros(cost.size, np.int32), 1,
                                          round_f32=True)
        got = view(ctx, cost.size, 1)
        assert np.array_equal(got[2], want[2])
        for k in (0, 1, 3):
            assert np.array_equal(got[k].astype(np.float64), want[k]), k
        assert not np.signbit(got[0]).any()


# below zero, and what is no number with the sign of each kind
@pytest.mark.parametrize("bits", [0xbf800000, 0x80000001, 0xff800000, 0x7fc00000, 0xffc00000])
def test_costs_below_zero_are_reported(ctx, bits):
    """Such a cost is not taken (a new node's counts as 0, an observed one changes nothing) and the stream status says so; all
    other costs of the call are."""
    from paper_2605_16637_amd import binding
    bad = np.array([bits], np.uint32).view(np.float32)[0]

    def reported():
        with pytest.raises(binding.HxError) as e:
            ctx.hx_stream_status()
        assert e.value.code == -1

    # 0 <- 1 <- 2 <- 3 and 1 <- 4; the leaf 3 is what everything above hangs on
    prow, pcol, wf = np.array([0, 0, 1, 2, 3, 4], np.int32), np.array([0, 1, 2, 1], np.int32), np.zeros(5, np.int32)

    def check(cost):
        want = o.critical_path_by_parents(prow, pcol, np.array(cost, np.float64), wf, 1, round_f32=True)
        got = view(ctx, 5, 1)
        assert np.array_equal(got[2], want[2])
        for k in (0, 1, 3):
            assert np.array_equal(got[k].astype(np.float64), want[k]), k

    ctx.hx_dag_reserve(8, 8, 1, 8)
    ctx.hx_dag_append(dev(prow), dev(pcol), dev(np.array([1, bad, 2, 4, 0.5], np.float32)), dev(wf))
    reported()
    check([1, 0, 2, 4, 0.5])
    ctx.hx_dag_set_cost(dev(np.array([1, 3, 0], np.int32)), dev(np.array([3, bad, 2], np.float32)))
    reported()
    check([2, 3, 2, 4, 0.5])
    ctx.hx_dag_set_cost(dev(np.array([3, 4], np.int32)), dev(np.array([np.inf, 0.0], np.float32)))       # without limit: a cost
    ctx.hx_stream_status()
    check([2, 3, 2, np.inf, 0])


# a node's parents beyond the second are raised three at a time: every remainder, one of them named twice, one not an earlier node
@pytest.mark.parametrize("parents", [2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 19, 20])
@pytest.mark.parametrize("odd", ["", "twice", "no parent"])
def test_append_of_a_node_with_parents(ctx, parents, odd):
    from paper_2605_16637_amd import binding
    rng = np.random.default_rng(parents)
    n0 = parents + 3                                         # parents of one child each, over them a root, beside them two others
    row = np.concatenate([[0, 0], np.arange(1, n0)]).astype(np.int32)
    col = np.zeros(n0 - 1, np.int32)
    cost = rng.uniform(0.1, 2.0, n0 + 2).astype(np.float32)
    up = 1 + rng.permutation(n0 - 1)[:parents].astype(np.int32)
    if odd == "twice":
        up[-1] = up[0]
    given, kept = up.copy(), up
    if odd == "no parent":
        given[parents // 2] = n0 + 5
        kept = np.delete(up, parents // 2)
    ctx.hx_dag_reserve(n0 + 2, 2 * n0 + 2 * parents, 1, 8)
    ctx.hx_dag_append(dev(row), dev(col), dev(cost[:n0]), dev(np.zeros(n0, np.int32)))
    # the node, and a child of it, in one batch
    ctx.hx_dag_append(dev(np.array([0, parents, parents + 1], np.int32)), dev(np.append(given, n0).astype(np.int32)), dev(cost[n0:]),
                      dev(np.zeros(2, np.int32)))
    if odd == "no parent":
        with pytest.raises(binding.HxError) as e:
            ctx.hx_stream_status()
        assert e.value.code == -3
    ctx.hx_stream_status()
    prow = np.concatenate([row, [n0 - 1 + kept.size, n0 + kept.size]]).astype(np.int32)
    pcol = np.concatenate([col, kept, [n0]]).astype(np.int32)
    for again in (False, True):
        want = o.critical_path_by_parents(prow, pcol, cost.astype(np.float64), np.zeros(n0 + 2, np.int32), 1, round_f32=True)
        got = view(ctx, n0 + 2, 1)
        assert np.array_equal(got[2], want[2])
        for k in (0, 1, 3):
            assert np.array_equal(got[k].astype(np.float64), want[k]), k
        cost[n0:] = [0.25, 7.0]
        ctx.hx_dag_set_cost(dev(np.array([n0, n0 + 1], np.int32)), dev(cost[n0:]))
        ctx.hx_stream_status()


# a walk that has ended goes on from the highest second parent above it: one for several nodes, each its own, some with nothing
# to raise, and a row of them, one walk along it up to and beyond the walk's 1024 steps
@pytest.mark.parametrize("kind", ["shared", "own", "some higher", "row"])
@pytest.mark.parametrize("above", [1, 2, 3, 4, 5, 8, 9])
def test_append_goes_on_from_second_parents(ctx, kind, above):
    rng = np.random.default_rng(above)
    if kind == "row":                                        # first parent the root, which the first child raises; second the node before
        n = {1: 3, 2: 5, 3: 64, 4: 1023, 5: 1024, 8: 1025, 9: 1500}[above] + 2
        parents, sizes = [[], [0]] + [[0, v - 1] for v in range(2, n)], [n]
    else:                                                    # rows over a root; on them a chain, each node a second parent at a row's end; below it a node
        rows, parents = above if kind == "own" else 1 if kind == "shared" else 2, [[]]
        for k in range(rows):
            for j in range(5):
                parents.append([0 if j == 0 else len(parents) - 1])
        ends = [5 * (k + 1) for k in range(rows)]
        for k in range(above):
            parents.append([len(parents) - 1 if k else 0, ends[(above - 1 - k) % rows]])
        parents.append([len(parents) - 1])
        n = len(parents)
        sizes = [n - 1, 1]
    row = np.cumsum([0] + [len(p) for p in parents]).astype(np.int32)
    col = np.array([u for p in parents for u in p], np.int32)
    cost = rng.uniform(0.5, 2.0, n).astype(np.float32)
    if kind == "some higher":
        sizes = [n - 1, 1, 1]
        row = np.append(row, row[-1] + 1).astype(np.int32)   # first a child of one of the second parents that no path through the chain exceeds
        col = np.append(col[:row[n - 1]], [ends[0], col[-1]]).astype(np.int32)
        cost = np.append(cost, cost[:1]).astype(np.float32)
        cost[n - 1] = 1000.0
        n += 1
    wf = np.zeros(n, np.int32)
    ctx.hx_dag_reserve(n, col.size, 1, n)
    v = 0
    for k in sizes:
        ctx.hx_dag_append(dev(row[v:v + k + 1] - row[v]), dev(col[row[v]:row[v + k]]), dev(cost[v:v + k]), dev(wf[v:v + k]))
        v += k
    for again in (False, True):
        ctx.hx_stream_status()
        want = o.critical_path_by_parents(row, col, cost.astype(np.float64), wf, 1, round_f32=True)
        got = view(ctx, n, 1)
        assert np.array_equal(got[2], want[2])
        for k in (0, 1, 3):
            assert np.array_equal(got[k].astype(np.float64), want[k]), k
        cost[n - 1] = 3.0
        ctx.hx_dag_set_cost(dev(np.array([n - 1], np.int32)), dev(cost[n - 1:]))


def wide_graph(kind):
    """Parent lists (row, col) of graphs whose nodes without children are few and whose nodes have several parents."""
    rng = np.random.default_rng(len(kind))
    if kind == "near parents":                               # 20 workflows of 1000 nodes, up to three parents among the eight before
        parents = [sorted(set((rng.integers(max(0, v - 8), v, 3)).tolist())) if v else [] for v in range(1000)]
        copies = 20
    else:                                                    # 20 of 40 layers of 10, all of a layer above all of the next
        parents = [list(range(v // 10 * 10 - 10, v // 10 * 10)) if v >= 10 else [] for v in range(400)]
        copies = 20
    size = len(parents)
    deg, one = np.array([len(p) for p in parents]), np.array([u for p in parents for u in p])
    row = np.concatenate([[0], np.cumsum(np.tile(deg, copies))]).astype(np.int32)
    return row, (one + size * np.arange(copies)[:, None]).astype(np.int32).reshape(-1), np.repeat(np.arange(copies, dtype=np.int32), size)


@pytest.mark.parametrize("kind", ["near parents", "layers"])
def test_observed_costs_where_few_nodes_have_no_children(ctx, kind):
    """New costs are carried up by every node of such a graph, not by its few leaves alone: their walks would visit all of it one after the
    other (54 and 8 ms here; appending the graph, where every node walks, takes 9.2 and 3.8)."""
    import torch
    row, col, wf = wide_graph(kind)
    n, n_wf = wf.size, int(wf.max()) + 1
    rng = np.random.default_rng(4)
    cost = rng.uniform(0.1, 2.0, n).astype(np.float32)
    ids = np.arange(0, n, 7, dtype=np.int32)
    new = rng.uniform(0.05, 3.0, ids.size).astype(np.float32)
    g = [dev(x) for x in (row, col, cost, wf, ids, new)]

    def ms(fn):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(); fn(); b.record()
        ctx.hx_stream_status()
        return a.elapsed_time(b)

    append, refresh = [], []
    for _ in range(3):
        ctx.hx_dag_reserve(n, col.size, n_wf, 2000)
        torch.cuda.synchronize()
        append.append(ms(lambda: ctx.hx_dag_append(*g[:4])))
        refresh.append(ms(lambda: ctx.hx_dag_set_cost(g[4], g[5])))
    cost[ids] = new
    want = o.critical_path_by_parents(row, col, cost.astype(np.float64), wf, n_wf, round_f32=True)
    got = view(ctx, n, n_wf)
    assert np.array_equal(got[2], want[2])
    for k in (0, 1, 3):
        assert np.array_equal(got[k].astype(np.float64), want[k]), k
    # with every node walking a refresh is the append without its first kernel: half as much again at most
    assert min(refresh) < 1.5 * min(append), (refresh, append)


@pytest.mark.parametrize("per_node", [1, 2, 3])
def test_observed_costs_of_a_large_graph(ctx, per_node):
    """More nodes than a refresh lets walk together: the nodes without children alone walk (up to two edges a node), or all do."""
    rng = np.random.default_rng(per_node)
    n_wf, size = 30000, 10
    n = n_wf * size
    rank = np.tile(np.arange(size), n_wf)
    deg = np.minimum(rank, per_node)
    row = np.zeros(n + 1, np.int32); row[1:] = np.cumsum(deg)
    first = np.repeat(np.arange(n) - rank, deg)              # a node's parents: among those before it in its workflow, some twice
    col = (first + (rng.random(first.size) * np.repeat(rank, deg)).astype(np.int64)).astype(np.int32)
    wf = np.repeat(np.arange(n_wf, dtype=np.int32), size)
    cost = rng.choice(np.array([0.0, 0.25, 1.0, 3.0], np.float32), n)
    ctx.hx_dag_reserve(n, col.size, n_wf, 16)
    ctx.hx_dag_append(dev(row), dev(col), dev(cost), dev(wf))
    for _ in range(2):
        ids = rng.choice(n, n // 3, replace=False).astype(np.int32)
        cost[ids] = rng.choice(np.array([0.0, 0.5, 2.0], np.float32), ids.size)
        ctx.hx_dag_set_cost(dev(ids), dev(cost[ids]))
        ctx.hx_stream_status()
        want = o.critical_path_revealed(row, col, cost.astype(np.float64), wf, n_wf, round_f32=True)
        got = view(ctx, n, n_wf)
        assert np.array_equal(got[2], want[2])
        for k in (0, 1, 3):
            assert np.array_equal(got[k].astype(np.float64), want[k]), k


def test_append_errors(ctx):
    from paper_2605_16637_amd import binding
    ctx.hx_dag_reserve(8, 8, 2, 4)
    with pytest.raises(binding.HxError) as e:            # beyond the reserved store
        ctx.hx_dag_append(dev(np.zeros(10, np.int32)), dev(np.zeros(0, np.int32)), dev(np.ones(9, np.float32)),
                          dev(np.zeros(9, np.int32)))
    assert e.value.code == -4
    # a parent that is not an earlier node
    ctx.hx_dag_append(dev(np.array([0, 1], np.int32)), dev(np.array([0], np.int32)), dev(np.ones(1, np.float32)),
                      dev(np.zeros(1, np.int32)))
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -3
    # a chain deeper than max_depth is no error: the walks do not go level by level
    ctx.hx_dag_reserve(16, 16, 1, 2)
    ctx.hx_dag_append(dev(np.array([0, 0, 1, 2, 3, 4, 5], np.int32)), dev(np.arange(5, dtype=np.int32)),
                      dev(np.ones(6, np.float32)), dev(np.zeros(6, np.int32)))
    ctx.hx_stream_status()
    rem, tail, level, hor = view(ctx, 6, 1)
    assert list(rem) == [6, 5, 4, 3, 2, 1] and list(level) == [5, 4, 3, 2, 1, 0] and list(hor) == [6]


def test_a_reserve_of_a_similar_size_begins_an_empty_graph(ctx):
    # 16 nodes, then 10 of the same store: as empty as a new one, and no larger than was asked for; then another store
    from paper_2605_16637_amd import binding
    for cap in (16, 10, 16, 40):
        ctx.hx_dag_reserve(cap, cap, 2, 4)
        with pytest.raises(binding.HxError) as e:
            ctx.hx_dag_append(dev(np.zeros(cap + 2, np.int32)), dev(np.zeros(0, np.int32)), dev(np.ones(cap + 1, np.float32)),
                              dev(np.zeros(cap + 1, np.int32)))
        assert e.value.code == -4
        cost = np.arange(1, 7, dtype=np.float32)
        ctx.hx_dag_append(dev(np.array([0, 0, 1, 2, 3, 4, 5], np.int32)), dev(np.arange(5, dtype=np.int32)), dev(cost),
                          dev(np.ones(6, np.int32)))
        ctx.hx_stream_status()
        rem, tail, level, hor = view(ctx, 6, 2)
        assert list(rem) == list(np.cumsum(cost[::-1])[::-1]) and list(level) == [5, 4, 3, 2, 1, 0] and list(hor) == [0, 21]
        ctx.hx_dag_set_cost(dev(np.array([5], np.int32)), dev(np.array([100.0], np.float32)))
        ctx.hx_stream_status()
        assert view(ctx, 6, 2)[3][1] == 115


def test_a_first_reserve_does_not_wait_for_other_streams():
    import torch
    from paper_2605_16637_amd import binding
    c = binding.Context(0)
    side, mine = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(side):
        torch.cuda._sleep(400_000_000)               # some 0.2 s
        done.record()
    with torch.cuda.stream(mine):
        c.hx_dag_reserve(1000, 1000, 10, 8)
        first = done.query()
        c.hx_dag_reserve(900, 900, 10, 8)            # the same arrays again: nothing may be at work on them
        second = done.query()
    assert not first and second
    c.hx_stream_status()
    c.close()


def chain_and_fan(n_chain, n_fan):
    """A chain 0 <- 1 <- ... and then one node whose parents are the last n_fan chain nodes."""
    rp = np.concatenate([[0], np.arange(n_chain), [n_chain - 1 + n_fan]]).astype(np.int32)       # node 0 has no parent
    col = np.concatenate([np.arange(n_chain - 1), np.arange(n_chain - n_fan, n_chain)]).astype(np.int32)
    return rp, col


def test_append_walks_that_hand_over_to_the_sweeps(ctx):
    """A walk is cut short when more than 16 grown parents wait at once, or after 1024 visited nodes; the rest
    goes level by level.  Both paths must still give the full recomputation, and too few sweeps are reported."""
    from paper_2605_16637_amd import binding
    rng = np.random.default_rng(12)
    for n_chain, n_fan, depth in ((60, 40, 64), (1500, 1, 1500)):
        n = n_chain + 1
        rp, col = chain_and_fan(n_chain, n_fan)
        cost = rng.uniform(0.5, 2.0, n).astype(np.float32)
        ctx.hx_dag_reserve(n + 4, col.size + 4, 1, depth)
        # the chain first, then the node with the many parents
        ctx.hx_dag_append(dev(rp[:n_chain + 1]), dev(col[:n_chain - 1]), dev(cost[:n_chain]), dev(np.zeros(n_chain, np.int32)))
        ctx.hx_stream_status()
        ctx.hx_dag_append(dev(np.array([0, n_fan], np.int32)), dev(col[n_chain - 1:]), dev(cost[n_chain:]), dev(np.zeros(1, np.int32)))
        ctx.hx_stream_status()
        want = o.critical_path_by_parents(rp, col, cost.astype(np.float64), np.zeros(n, np.int32), 1, round_f32=True)
        got = view(ctx, n, 1)
        assert np.array_equal(got[2], want[2])
        for k in (0, 1, 3):
            assert np.array_equal(got[k].astype(np.float64), want[k]), k
    # the 1500-deep chain with room for 3 sweeps only: the cut walk cannot be finished, and says so
    rp, col = chain_and_fan(1500, 1)
    ctx.hx_dag_reserve(1600, 1600, 1, 3)
    ctx.hx_dag_append(dev(rp[:1501]), dev(col[:1499]), dev(np.ones(1500, np.float32)), dev(np.zeros(1500, np.int32)))
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -4


@pytest.mark.parametrize("C", [900, 5000, 200000])      # one launch (small rounds); two launches, few and many workgroups
def test_commit_matches_oracle(ctx, C):
    import torch
    from paper_2605_16637_amd import binding
    rng = np.random.default_rng(6)
    P, D = 37, 53
    L, O = synth.gen_lengths(rng, C)
    bp = rng.integers(-1, P, C).astype(np.int32)
    bd = np.where(bp < 0, -1, rng.integers(0, D, C)).astype(np.int32)
    st = [rng.integers(0, 20000, P).astype(np.int32), rng.integers(0, 300000, D).astype(np.int32),
          rng.integers(0, 200, D).astype(np.int32), rng.integers(0, 20000, D).astype(np.int32)]
    dr = [rng.integers(0, 80 * C, P).astype(np.int32), rng.integers(0, 6 * C, D).astype(np.int32),
          rng.integers(0, 40 * C, D).astype(np.int32)]
    want = o.commit(L, O, bp, bd, *st, *dr)
    assert want[4] == 0
    g = [dev(x.copy()) for x in st]
    calls = binding.to_device(dict(n=C, L_in=L, L_out=O))
    ctx.hx_commit(calls, dev(bp), dev(bd), g[0], g[1], g[2], g[3], dev(dr[0]), dev(dr[1]), dev(dr[2]))
    ctx.hx_stream_status()
    for got, w in zip(g, want[:4]):
        assert np.array_equal(got.cpu().numpy(), w)
    # overflow and a placement outside the pool are reported
    big = binding.to_device(dict(n=2, L_in=np.array([2**30, 2**30], np.int32), L_out=np.array([16, 16], np.int32)))
    g = [dev(np.zeros(1, np.int32)) for _ in range(4)]
    ctx.hx_commit(big, dev(np.zeros(2, np.int32)), dev(np.zeros(2, np.int32)), *g)
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -7
    ctx.hx_commit(big, dev(np.array([3, 0], np.int32)), dev(np.zeros(2, np.int32)), *g)
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -6


# where the commit's kernel or its workgroups change (2048 and 8192 calls), more instances on one side than a workgroup has
# threads, and placements that all meet on few instances (hot) or none
@pytest.mark.parametrize("C,P,D,hot", [(512, 256, 256, 1), (513, 256, 256, 1), (513, 257, 256, 1), (2049, 256, 256, 1), (2049, 256, 257, 1),
                                        (1, 1, 1, 0), (2048, 5, 1024, 0), (2049, 1024, 3, 0), (2049, 4, 4, 1), (8192, 600, 513, 0),
                                       (8193, 64, 64, 1), (8193, 1024, 1024, 0), (0, 600, 700, 0)])
def test_commit_at_the_lines_between_its_kernels(ctx, C, P, D, hot):
    from paper_2605_16637_amd import binding
    rng = np.random.default_rng(C + P)
    L, O = synth.gen_lengths(rng, C)
    bp = rng.integers(-1, min(P, 2) if hot else P, C).astype(np.int32)
    bd = rng.integers(-1, min(D, 2) if hot else D, C).astype(np.int32)         # one side alone keeps a call queued
    st = [rng.integers(0, 20000, P).astype(np.int32), rng.integers(0, 300000, D).astype(np.int32),
          rng.integers(0, 200, D).astype(np.int32), rng.integers(0, 20000, D).astype(np.int32)]
    for dr in ([rng.integers(0, 80 * C + 9, n).astype(np.int32) for n in (P, D, D)], [np.zeros(n, np.int32) for n in (P, D, D)]):
        want = o.commit(L, O, bp, bd, *st, *dr)
        assert want[4] == 0
        g = [dev(x.copy()) for x in st]
        drains = [dev(x) for x in dr] if dr[0].any() else [None] * 3          # no drains: NULL
        ctx.hx_commit(binding.to_device(dict(n=C, L_in=L, L_out=O)), dev(bp), dev(bd), *g, *drains)
        ctx.hx_stream_status()
        for got, w in zip(g, want[:4]):
            assert np.array_equal(got.cpu().numpy(), w)


# One instance on a side, so that all calls of a wavefront meet there and their lengths are added by halves of 16 bits: lengths around
# the carry from one to the other, whole wavefronts, ragged ones, one alone; rounds of either commit kernel
@pytest.mark.parametrize("C", [1, 2, 63, 64, 65, 128, 2047, 2048, 2049, 8192, 16384])
@pytest.mark.parametrize("P,D", [(1, 1), (1, 3), (3, 1), (3, 3)])
def test_commit_of_long_calls_on_one_instance(ctx, C, P, D):
    from paper_2605_16637_amd import binding
    rng = np.random.default_rng(C + 10 * P + D)
    L, O = (rng.choice(np.array([0, 1, 65534, 65535, 65536, 65537], np.int32), C) for _ in range(2))
    for x in (L, O):
        x[rng.integers(0, C, 4)] = [1 << 20, (1 << 20) - 1, 3 << 16, 1 << 17]
    assert int(L.sum(dtype=np.int64)) + int(O.sum(dtype=np.int64)) < 2**31 - 4096        # no counter overflows
    # where there are three instances: all but some calls on the last
    bp, bd = (np.where(rng.random(C) < 0.02, rng.integers(-1, n, C), n - 1).astype(np.int32) for n in (P, D))
    st = [rng.integers(0, 999, n).astype(np.int32) for n in (P, D, D, D)]
    want = o.commit(L, O, bp, bd, *st, *[np.zeros(n, np.int32) for n in (P, D, D)])
    assert want[4] == 0
    g = [dev(x.copy()) for x in st]
    ctx.hx_commit(binding.to_device(dict(n=C, L_in=L, L_out=O)), dev(bp), dev(bd), *g)
    ctx.hx_stream_status()
    for got, w in zip(g, want[:4]):
        assert np.array_equal(got.cpu().numpy(), w)


# sweeps inside a workgroup's slice and over the whole graph: a workflow that fills a slice or does not fit one, more successors
# than a node has slots, rows at the very end of the id array, an edge into another slice, nodes of no workflow, and
# two graphs in a row (what the workgroups share has to be clear again)
@pytest.mark.parametrize("kind", ["full slice", "too large", "many successors", "few edges", "across", "no workflow", "empty workflows"])
def test_sweeps_by_slice_and_over_the_whole_graph(ctx, kind):
    rng = np.random.default_rng(sum(map(ord, kind)))
    sizes = {"full slice": [1024, 3, 1021], "too large": [700, 1025, 40], "many successors": [90, 64], "few edges": [3, 1],
             "across": [30] * 900, "no workflow": [50, 50], "empty workflows": [0, 5, 0, 0, 7, 0]}[kind]
    n = int(np.sum(sizes))
    wf_ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    succ = [[] for _ in range(n)]
    for a, b in zip(wf_ptr[:-1], wf_ptr[1:]):
        order = a + rng.permutation(b - a)                  # any numbering: edges go forward along `order`
        for i in range(b - a):
            later = order[i + 1:]
            if later.size and rng.random() < 0.85:
                many = 12 if kind == "many successors" else 3
                near = later[:40]
                succ[order[i]] = list(rng.choice(near, min(near.size, int(rng.integers(1, many + 1))), replace=False))
    if kind == "few edges":
        succ = [[2], [], [], []]
    if kind == "across":
        for k in range(5):                                   # whole workflows hang on later ones, wherever these are staged
            succ[int(wf_ptr[10 * k + 1] - 1)].append(int(wf_ptr[600 + 7 * k]))
    if kind == "no workflow":
        wf_ptr = np.array([10, 50, 90], np.int32)            # the first and the last ten nodes belong to none
    deg = np.array([len(x) for x in succ])
    row = np.zeros(n + 1, np.int32); row[1:] = np.cumsum(deg)
    col = np.array([u for x in succ for u in sorted(x)], np.int32)
    cost32 = rng.uniform(0.1, 2.0, n).astype(np.float32)
    want = o.critical_path(row, col, cost32.astype(np.float64), wf_ptr, round_f32=True)
    for _ in range(2):
        assert_cp_bit_exact(gpu_cp(ctx, row, col, cost32, wf_ptr, max_sweeps=int(want[2].max()) + 2), want)
    assert_cp_bit_exact(gpu_cp(ctx, row, col, cost32, wf_ptr, max_sweeps=4000), want)


# the sweeps over the whole graph at the sizes where they change: one workgroup or several, nodes kept in registers from sweep
# to sweep or read again (more than 4 per thread of 256 workgroups of 512), horizons by 16 lanes or by a wavefront;
# successors anywhere, or a chain of workflows each of which hangs on the next
@pytest.mark.parametrize("n_wf,size", [(7, 3), (25, 20), (26, 20), (300, 20), (60, 200), (26300, 20)])
@pytest.mark.parametrize("kind", ["anywhere", "chain of workflows", "one workflow beside"])
def test_sweeps_over_the_whole_graph_at_its_sizes(ctx, n_wf, size, kind):
    rng = np.random.default_rng(n_wf + size)
    n = n_wf * size
    if kind == "one workflow beside":                        # a workflow that fits no slice: everything from the beginning
        n += 1100
    wf_ptr = np.append(np.arange(n_wf) * size, [n_wf * size, n][n > n_wf * size:]).astype(np.int32)
    at = rng.permutation(n) if kind == "anywhere" else np.arange(n)
    i = np.arange(n - 1)
    deg = rng.integers(0, 4, n - 1)                          # up to three successors, later along `at`
    src = np.repeat(i, deg)
    dst = src + (rng.integers(n // 12 + 1, n // 6 + 2, src.size) if kind == "anywhere" else rng.integers(1, 4, src.size))
    keep = dst < n
    if kind != "anywhere":
        keep &= np.minimum(src // size, n_wf) == np.minimum(dst // size, n_wf)      # inside a workflow
    src, dst = src[keep], dst[keep]
    if kind == "chain of workflows":
        last = np.arange(1, min(n_wf, 12)) * size - 1
        src, dst = np.append(src, last), np.append(dst, last + 1)
    edges = np.unique(np.stack([at[src], at[dst]], 1), axis=0)
    row = np.zeros(n + 1, np.int32); row[1:] = np.cumsum(np.bincount(edges[:, 0], minlength=n))
    col = edges[:, 1].astype(np.int32)
    cost32 = rng.uniform(0.1, 2.0, n).astype(np.float32)
    want = o.critical_path(row, col, cost32.astype(np.float64), wf_ptr, round_f32=True)
    limit = int(want[2].max()) + 2
    assert 2 < limit < 2000
    for _ in range(2):
        assert_cp_bit_exact(gpu_cp(ctx, row, col, cost32, wf_ptr, max_sweeps=limit), want)


def test_sweeps_report_a_cycle_between_slices(ctx):
    from paper_2605_16637_amd import binding
    n_wf, size = 400, 5
    n = n_wf * size
    # every workflow a chain; the first hangs on the last and the last on the first
    succ = [[v + 1] if (v + 1) % size else [] for v in range(n)]
    succ[size - 1], succ[n - 1] = [n - size], [0]
    row = np.zeros(n + 1, np.int32); row[1:] = np.cumsum([len(x) for x in succ])
    col = np.array([u for x in succ for u in x], np.int32)
    cost32 = np.ones(n, np.float32)
    gpu_cp(ctx, row, col, cost32, np.arange(n_wf + 1) * size, max_sweeps=50, check=False)
    with pytest.raises(binding.HxError) as e:
        ctx.hx_stream_status()
    assert e.value.code == -3
    # without the way back it is a graph of depth 9
    row[n:] -= 1
    want = o.critical_path(row, col[:-1], cost32.astype(np.float64), np.arange(n_wf + 1) * size, round_f32=True)
    assert want[2].max() == 2 * size - 1
    assert_cp_bit_exact(gpu_cp(ctx, row, col[:-1], cost32, np.arange(n_wf + 1) * size, max_sweeps=2 * size + 1), want)


# The workgroups of the sweeps over the whole graph do not come together: with no polls all but the last to arrive give up at
# once, and the last to leave does the graph alone.  Afterwards the shared words are clear: the next graph, with the usual
# patience, comes out right, and so does one that the slices finish.
@pytest.mark.parametrize("kind", ["anywhere", "chain of workflows", "one workflow beside", "no workflows", "cycle"])
def test_sweeps_whose_workgroups_do_not_meet(kind):
    from paper_2605_16637_amd import binding
    c = binding.Context(0)
    assert c.lib.hx_test_sweep_polls(c._ctx, -1) == -1
    rng = np.random.default_rng(len(kind))
    n_wf, size = 200, 30
    n = n_wf * size
    if kind == "one workflow beside":
        n += 1500
    wf_ptr = np.append(np.arange(n_wf) * size, [n_wf * size, n][n > n_wf * size:]).astype(np.int32)
    at = rng.permutation(n) if kind == "anywhere" else np.arange(n)
    src = np.repeat(np.arange(n - 1), rng.integers(0, 4, n - 1))
    dst = src + (rng.integers(n // 12 + 1, n // 6 + 2, src.size) if kind == "anywhere" else rng.integers(1, 4, src.size))
    keep = dst < n
    if kind != "anywhere":
        keep &= np.minimum(src // size, n_wf) == np.minimum(dst // size, n_wf)
    src, dst = src[keep], dst[keep]
    inside = src.size
    if kind in ("chain of workflows", "cycle"):              # the first eight workflows, first node to first node
        src, dst = np.append(src, np.arange(7) * size), np.append(dst, np.arange(1, 8) * size)

    def graph(src, dst):
        edges = np.unique(np.stack([at[src], at[dst]], 1), axis=0)
        row = np.zeros(n + 1, np.int32); row[1:] = np.cumsum(np.bincount(edges[:, 0], minlength=n))
        return row, edges[:, 1].astype(np.int32)

    row, col = graph(src, dst)
    if kind == "no workflows":
        wf_ptr = np.zeros(1, np.int32)
    cost32 = rng.uniform(0.1, 2.0, n).astype(np.float32)
    if kind == "cycle":
        c.lib.hx_test_sweep_polls(c._ctx, 0)
        looped = graph(np.append(src, 7 * size), np.append(dst, 0))      # and back again: reported, also by the last one alone
        gpu_cp(c, *looped, cost32, wf_ptr, max_sweeps=60, check=False)
        with pytest.raises(binding.HxError) as e:
            c.hx_stream_status()
        assert e.value.code == -3
    want = o.critical_path(row, col, cost32.astype(np.float64), wf_ptr, round_f32=True)
    limit = int(want[2].max()) + 2
    for polls in (0, 0, 1 << 18, 3, 1 << 18):
        assert c.lib.hx_test_sweep_polls(c._ctx, polls) == 0
        assert_cp_bit_exact(gpu_cp(c, row, col, cost32, wf_ptr, max_sweeps=limit), want)
    if kind == "chain of workflows":
        row, col = graph(src[:inside], dst[:inside])
        want = o.critical_path(row, col, cost32.astype(np.float64), wf_ptr, round_f32=True)
        assert_cp_bit_exact(gpu_cp(c, row, col, cost32, wf_ptr, max_sweeps=limit), want)
    c.close()
