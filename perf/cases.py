"""The work a user of the placement search has it do, as cases that can be timed.

Each case is one pass through the public entry points of ``binding.Context`` on
device-resident inputs: a scheduling round, a stretch of a live system's rounds,
the cost tensor on request, the horizon refresh of a large workflow set, the
decode stage, and the two planners of small queues.  Inputs are the seeded
synthetic rounds of ``synth``; sizes are those of its workloads, of the tests
and of the benchmark, with ragged ones between them.
"""
import math
import zlib

import numpy as np
import torch

from paper_2605_16637_amd import binding, synth

DEV = "cuda:0"


def listed():
    return [
        # the round of a small deployment (64 calls on 4 + 4 instances, 8 short workflows): what a scheduler invocation costs at least
        dict(name="round tiny", kind="round", calls=64, prefill=4, decode=4, types=2, workflows=8, small_dags=True,
             near_capacity=False, one_call=True),
        # a busy cluster's round: 4096 ready calls of 1000 agentic workflows
        dict(name="round mid", kind="round", calls=4096, prefill=64, decode=64, types=4, workflows=1000, small_dags=False,
             near_capacity=False, one_call=True),
        # a large pool near its KV capacity, where most of the time is the search
        dict(name="round large", kind="round", calls=16384, prefill=256, decode=256, types=8, workflows=4096, small_dags=False,
             near_capacity=True, one_call=True),
        # a ragged pool, the round made of its separate library calls (horizons, search with the ratio, commit)
        dict(name="round ragged three calls", kind="round", calls=1537, prefill=47, decode=101, types=5, workflows=389,
             small_dags=False, near_capacity=True, one_call=False),
        # a live system: what is live is appended to an empty store, then consecutive rounds reveal, score and commit, then
        # observed costs replace estimates and the urgencies of the last round are formed again
        dict(name="stream session", kind="stream", live=20000, calls=32768, prefill=512, decode=512, types=8, rounds=8),
        # every candidate's cost and the feasibility mask written out, then the selection over the tensor (studies, other policies)
        dict(name="cost tensor and select", kind="tensor", calls=4096, prefill=64, decode=64, types=4, near_capacity=False),
        # horizons of a very large workflow set from scratch: standalone costs, then the single-pass critical path
        dict(name="horizons of 100000 workflows", kind="horizons", workflows=100000, sweeps=0),
        # the critical path of graphs in arbitrary numbering: level-synchronous sweeps up to the depth limit
        dict(name="horizons any numbering", kind="horizons", workflows=1000, sweeps=14),
        # the decode stage of a large queue: one scoring pass with half the calls locked, then the one-pass ordering
        dict(name="decode pass", kind="decode", calls=16384, decode=256, types=8, resident=112, planned=12),
        # the decode stage's recomputing greedy on a small queue
        dict(name="decode plan", kind="decode_plan", calls=256, decode=32, types=4, resident=24, planned=4),
        # the recomputing greedy of small queues: a pool of the size the paper serves, and the larger of the benchmark's
        dict(name="plan 64 on 8+8", kind="plan", calls=64, prefill=8, decode=8, types=3),
        dict(name="plan 256 on 64+64", kind="plan", calls=256, prefill=64, decode=64, types=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["round", "round", "round", "stream", "tensor", "horizons", "decode", "decode_plan", "plan"])
    types = rng.randint(1, 8)
    if kind == "round":
        calls = _log(rng, 16, 16384)
        return dict(kind=kind, calls=calls, prefill=_log(rng, 2, 256), decode=_log(rng, 2, 256), types=types,
                    workflows=max(4, calls // rng.randint(3, 8)), small_dags=rng.random() < 0.3,
                    near_capacity=rng.random() < 0.5, one_call=rng.random() < 0.6)
    if kind == "stream":
        live = _log(rng, 256, 16000)
        return dict(kind=kind, live=live, calls=_log(rng, live, 2 * live), prefill=_log(rng, 16, 400), decode=_log(rng, 16, 400),
                    types=types, rounds=8)
    if kind == "tensor":
        prefill, decode = _log(rng, 4, 128), _log(rng, 4, 128)
        return dict(kind=kind, calls=_log(rng, 16, min(4096, 16000000 // (prefill * decode))), prefill=prefill, decode=decode,
                    types=types, near_capacity=rng.random() < 0.5)
    if kind == "horizons":
        sweeps = rng.random() < 0.3
        return dict(kind=kind, workflows=_log(rng, 50, 1000 if sweeps else 90000), sweeps=14 if sweeps else 0)
    if kind == "decode":
        return dict(kind=kind, calls=_log(rng, 48, 20000), decode=_log(rng, 4, 256), types=types, resident=rng.randint(10, 112),
                    planned=rng.randint(1, 12))
    if kind == "decode_plan":
        return dict(kind=kind, calls=_log(rng, 8, 256), decode=_log(rng, 2, 32), types=types, resident=rng.randint(8, 24),
                    planned=rng.randint(1, 4))
    return dict(kind=kind, calls=_log(rng, 8, 256), prefill=_log(rng, 2, 64), decode=_log(rng, 2, 64), types=types)


# ---- what a user's program has in hand -------------------------------------------------


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _i32(n):
    return torch.empty(n, dtype=torch.int32, device=DEV)


def _f32(n):
    return torch.empty(n, dtype=torch.float32, device=DEV)


# Arrays over the nodes of a graph are kept at the most nodes it can have, as a serving program keeps them: the library
# writes the nodes there are, the rest stays zero.
def _zeros(n, dtype=torch.float32):
    return torch.zeros(n, dtype=dtype, device=DEV)


def _rng_seed(case, seed):
    shape = ",".join("%s=%s" % (k, case[k]) for k in sorted(case) if k != "name")
    return (zlib.crc32(shape.encode()) << 31) + int(seed)


def _pool_state(pre, dec):
    return dict(backlog_tok=pre["backlog_tok"], used_tok=dec["used_tok"], batch=dec["batch"], qd_tok=dec["qd_tok"])


def _drains(L_in, L_out, P, D):
    """Per-round drains of what a round adds, so that the pool stays in its regime from round to round."""
    Ls, Os = int(L_in.sum()), int(L_out.sum())
    return (_dev(np.full(P, Ls // P, np.int32)), _dev(np.full(D, Os // D, np.int32)), _dev(np.full(D, (Ls + Os) // D, np.int32)))


def _round_inputs(case, seed, workflows, small_dags):
    lo, hi, fan, depth, p2, recency = (4, 12, 3, 5, 0.3, 0.5) if small_dags else (10, 30, 4, 12, 0.4, 1.0)
    return synth.make_round("mid", _rng_seed(case, seed), n_wf=workflows, size_lo=lo, size_hi=hi, fanout_max=fan, depth_max=depth,
                            p_second=p2, recency=recency, C=case["calls"], P=case["prefill"], D=case["decode"], T=case["types"],
                            near_capacity=case["near_capacity"])


def _prepare_round(case, seed):
    r = _round_inputs(case, seed, case["workflows"], case["small_dags"])
    ctx, d, n = binding.Context(0), r.dag, case["calls"]
    calls, pre, dec, links = (binding.to_device(x) for x in (r.calls, r.pre, r.dec, r.links))
    tF, tB = _dev(r.types["flops"]), _dev(r.types["hbm_bw"])
    room = d.n_wf * (12 if case["small_dags"] else 30)
    g = dict(succ_row_ptr=_dev(d.succ_row_ptr), succ_col_idx=_dev(d.succ_col), wf_ptr=_dev(d.wf_ptr), L_in=_dev(d.L_in),
             L_out=_dev(d.L_out), node_cost=_zeros(room), rem=_zeros(room), tail=_zeros(room), level=_zeros(room, torch.int32),
             horizon=_f32(d.n_wf))
    bp, bd, bc, ratio = _i32(n), _i32(n), _f32(n), _f32(n)
    drain_p, drain_q, release = _drains(r.calls["L_in"], r.calls["L_out"], case["prefill"], case["decode"])

    def one_call():
        ctx.hx_round(r.model, calls, pre, dec, links, bp, bd, bc, ratio=ratio, type_flops=tF, type_hbm_bw=tB,
                     drain_prefill=drain_p, drain_decode_q=drain_q, release_tok=release, graph=g)

    def three_calls():
        ctx.hx_horizons(r.model, g["succ_row_ptr"], g["succ_col_idx"], g["L_in"], g["L_out"], tF, tB, links, g["wf_ptr"],
                        g["node_cost"], g["rem"], g["tail"], g["level"], g["horizon"])
        ctx.hx_score_placements(r.model, calls, pre, dec, links, tail=g["tail"], horizon=g["horizon"],
                                best_p=bp, best_d=bd, best_cost=bc, ratio=ratio)
        ctx.hx_commit(calls, bp, bd, pre["backlog_tok"], dec["used_tok"], dec["batch"], dec["qd_tok"], drain_p, drain_q, release)

    # a scheduling loop works on the same buffers round after round and marshals its arguments once
    go = ctx.prepare(one_call if case["one_call"] else three_calls)
    out = dict(best_p=bp, best_d=bd, best_cost=bc, ratio=ratio, **_pool_state(pre, dec),
               **{k: g[k] for k in ("node_cost", "rem", "tail", "level", "horizon")})
    return dict(ctx=ctx, run=lambda: (go(), out)[1], keep=(calls, pre, dec, links, tF, tB, g, drain_p, drain_q, release))


def _prepare_stream(case, seed):
    seed = _rng_seed(case, seed)
    rng, gen = np.random.default_rng(seed), synth.StreamGen(seed, case["live"])
    P, D, C = case["prefill"], case["decode"], case["calls"]
    L0, O0 = synth.gen_lengths(rng, 20000)
    types, links, pre, dec = synth.gen_pool(rng, P, D, case["types"], L0, O0, near_capacity=True)
    ctx = binding.Context(0)
    links, pre, dec = binding.to_device(links), binding.to_device(pre), binding.to_device(dec)
    tF, tB = _dev(types["flops"]), _dev(types["hbm_bw"])
    pool0 = {k: v.clone() for k, v in _pool_state(pre, dec).items()}
    # what is live when the session begins (three rounds' worth of reveals), then the rounds
    live = []
    for b in (gen.next_batch() for _ in range(3)):
        live.append(dict(prow=_dev(b["parent_row_ptr"]), pcol=_dev(b["parent_col"]), wf=_dev(b["wf"]), L_in=_dev(b["L_in"]),
                         L_out=_dev(b["L_out"]), cost=_f32(b["n_new"])))
    rounds = []
    for b in (gen.next_batch() for _ in range(case["rounds"])):
        n = b["n_new"]
        pick = np.sort(rng.choice(n, min(C, n), replace=False)).astype(np.int32)
        k = int(pick.size)
        rounds.append(dict(
            n_wf=b["n_wf_total"], prow=_dev(b["parent_row_ptr"]), pcol=_dev(b["parent_col"]), wf=_dev(b["wf"]),
            L_in=_dev(b["L_in"]), L_out=_dev(b["L_out"]), cost=_zeros(gen.max_new * case["live"]),
            calls=dict(n=k, L_in=_dev(b["L_in"][pick]), L_out=_dev(b["L_out"][pick]), node=_dev(b["ids"][pick]),
                       wf=_dev(b["wf"][pick]), elapsed=_dev(rng.uniform(0, 30, k).astype(np.float32))),
            drains=_drains(b["L_in"][pick], b["L_out"][pick], P, D),
            best_p=_i32(k), best_d=_i32(k), best_cost=_f32(k), ratio=_f32(k)))
    n_seen = int(rng.integers(gen.n_nodes // 100, gen.n_nodes // 50 + 2))
    seen = _dev(np.sort(rng.choice(gen.n_nodes, n_seen, replace=False)).astype(np.int32))
    seen_cost = _dev(rng.uniform(0.5, 20.0, n_seen).astype(np.float32))
    n_edges = sum(int(b["pcol"].numel()) for b in live + rounds)
    last, late = rounds[-1], _f32(rounds[-1]["calls"]["n"])

    def session():
        ctx.hx_dag_reserve(gen.n_nodes, n_edges, gen.n_wf, 32)
        for b in live:
            ctx.hx_node_cost(synth.MODEL, b["L_in"], b["L_out"], tF, tB, links, b["cost"])
            ctx.hx_dag_append(b["prow"], b["pcol"], b["cost"], b["wf"])
        for b in rounds:
            ctx.hx_round(synth.MODEL, b["calls"], pre, dec, links, b["best_p"], b["best_d"], b["best_cost"], ratio=b["ratio"],
                         n_wf=b["n_wf"], parent_row_ptr=b["prow"], parent_col_idx=b["pcol"], new_L_in=b["L_in"],
                         new_L_out=b["L_out"], new_wf=b["wf"], new_cost=b["cost"], type_flops=tF, type_hbm_bw=tB,
                         drain_prefill=b["drains"][0], drain_decode_q=b["drains"][1], release_tok=b["drains"][2])
        ctx.hx_dag_set_cost(seen, seen_cost)

    go = ctx.prepare(session)
    out = dict(late=late, **_pool_state(pre, dec))
    for i, b in enumerate(rounds):
        for k in ("best_p", "best_d", "best_cost", "ratio", "cost"):
            out["%s %d" % (k, i)] = b[k]

    def run():
        for k, v in _pool_state(pre, dec).items():      # the session's pool as it was found
            v.copy_(pool0[k])
        go()
        _, tail, _, horizon, _ = ctx.hx_dag_view(last["n_wf"])
        ctx.hx_urgency(last["calls"], last["best_cost"], tail, horizon, late)
        return out

    return dict(ctx=ctx, run=run, keep=(links, pre, dec, tF, tB, live, rounds, seen, seen_cost))


def _prepare_tensor(case, seed):
    r = _round_inputs(case, seed, max(1, case["calls"] // 4), False)
    ctx, n, P, D = binding.Context(0), case["calls"], case["prefill"], case["decode"]
    calls, pre, dec, links = (binding.to_device(x) for x in (r.calls, r.pre, r.dec, r.links))
    rng = np.random.default_rng(_rng_seed(case, seed))
    tail = _dev(rng.uniform(0, 5, r.dag.n_nodes).astype(np.float32))
    horizon = _dev(rng.uniform(10, 60, r.dag.n_wf).astype(np.float32))
    cost, feas = _f32(n * P * D), torch.empty(n * D, dtype=torch.uint8, device=DEV)
    bp, bd, bc, ratio = _i32(n), _i32(n), _f32(n), _f32(n)

    def run():
        ctx.hx_score_placements(r.model, calls, pre, dec, links, cost=cost, feas=feas)
        ctx.hx_select(n, P, D, cost, bp, bd, bc, calls=calls, tail=tail, horizon=horizon, ratio=ratio)
        return dict(cost=cost, feas=feas, best_p=bp, best_d=bd, best_cost=bc, ratio=ratio)

    return dict(ctx=ctx, run=run)


def _prepare_horizons(case, seed):
    rng = np.random.default_rng(_rng_seed(case, seed))
    shape = (10, 30, 4, 12, 0.4, 1.0) if case["sweeps"] else (8, 32, 4, 32, 0.84, 2.0)
    d = synth.gen_dag(rng, case["workflows"], *shape)
    types = synth.type_table(4)
    ctx, links = binding.Context(0), binding.to_device(synth.link_table(types))
    tF, tB = _dev(types["flops"]), _dev(types["hbm_bw"])
    row, col, wf = d.succ_row_ptr, d.succ_col, d.wf_ptr
    L_in, L_out = d.L_in, d.L_out
    if case["sweeps"]:
        # the nodes of every workflow renumbered: successors lie anywhere
        n = d.n_nodes
        new = np.lexsort((rng.random(n), d.wf_of_node))            # a random order inside each workflow
        to = np.empty(n, np.int64)
        to[new] = np.arange(n)
        src, dst = to[np.repeat(np.arange(n), np.diff(row))], to[col]
        order = np.lexsort((dst, src))
        row = np.zeros(n + 1, np.int32)
        row[1:] = np.cumsum(np.bincount(src, minlength=n))
        col = dst[order].astype(np.int32)
        L_in, L_out = L_in[new], L_out[new]
    row, col, wf, L_in, L_out = (_dev(x) for x in (row, col, wf, L_in, L_out))
    room = d.n_wf * shape[1]
    cost, rem, tail, level, horizon = _zeros(room), _zeros(room), _zeros(room), _zeros(room, torch.int32), _f32(d.n_wf)

    def run():
        ctx.hx_node_cost(synth.MODEL, L_in, L_out, tF, tB, links, cost)
        ctx.hx_critical_path(row, col, cost, wf, rem, tail, level, horizon, max_sweeps=case["sweeps"])
        return dict(cost=cost, rem=rem, tail=tail, level=level, horizon=horizon)

    return dict(ctx=ctx, run=run)


def _decode_inputs(case, seed, stride):
    r, lock, iv = synth.make_decode_round("decode_mid", _rng_seed(case, seed), n_wf=max(4, case["calls"] // 4), Q=case["calls"],
                                          D=case["decode"], T=case["types"], stride=case["resident"] + case["planned"],
                                          n_resident=case["resident"], n_planned=case["planned"])
    D, K0 = case["decode"], iv["stride"]
    out = dict(stride=stride, count=_dev(iv["count"]))
    for k in ("start", "end", "tok"):
        a = np.zeros((D, stride), iv[k].dtype)
        a[:, :K0] = iv[k].reshape(D, K0)
        out[k] = _dev(a.reshape(-1))
    rng = np.random.default_rng(_rng_seed(case, seed))
    tail = _dev(rng.uniform(0, 5, r.dag.n_nodes).astype(np.float32))
    horizon = _dev(rng.uniform(10, 60, r.dag.n_wf).astype(np.float32))
    return binding.to_device(r.calls), _dev(lock), binding.to_device(r.dec), out, tail, horizon


def _prepare_decode(case, seed):
    queue, lock, dec, iv, tail, horizon = _decode_inputs(case, seed, case["resident"] + case["planned"] + 4)
    ctx, n = binding.Context(0), case["calls"]
    bd, bs, bc, ratio, rank = _i32(n), _f32(n), _f32(n), _f32(n), _i32(n)

    def run():
        ctx.hx_decode_score(synth.MODEL, queue, lock, dec, iv, bd, bs, bc, tail=tail, horizon=horizon, ratio=ratio)
        ctx.hx_rank(ratio, rank)
        return dict(best_d=bd, best_start=bs, best_cost=bc, ratio=ratio, rank=rank)

    return dict(ctx=ctx, run=run)


def _prepare_decode_plan(case, seed):
    queue, lock, dec, iv, tail, horizon = _decode_inputs(case, seed, min(case["resident"] + case["planned"] + case["calls"], 140))
    ctx, n, count0 = binding.Context(0), case["calls"], iv["count"].clone()
    bd, bs, bc, ratio, rank = _i32(n), _f32(n), _f32(n), _f32(n), _i32(n)

    def run():
        iv["count"].copy_(count0)               # every plan starts from the snapshot
        ctx.hx_decode_plan_greedy(synth.MODEL, queue, lock, dec, iv, tail, horizon, bd, bs, bc, ratio, rank)
        return dict(best_d=bd, best_start=bs, best_cost=bc, ratio=ratio, rank=rank, count=iv["count"])

    return dict(ctx=ctx, run=run)


def _prepare_plan(case, seed):
    r = _round_inputs(dict(case, near_capacity=False), seed, max(4, case["calls"] // 4), False)
    ctx, n, P, D = binding.Context(0), case["calls"], case["prefill"], case["decode"]
    calls, pre, dec, links = (binding.to_device(x) for x in (r.calls, r.pre, r.dec, r.links))
    rng = np.random.default_rng(_rng_seed(case, seed))
    tail = _dev(rng.uniform(0, 5, r.dag.n_nodes).astype(np.float32))
    horizon = _dev(rng.uniform(10, 60, r.dag.n_wf).astype(np.float32))
    bp, bd, bc, ratio, rank = _i32(n), _i32(n), _f32(n), _f32(n), _i32(n)
    backlog, used, batch, qd = _i32(P), _i32(D), _i32(D), _i32(D)

    def run():
        ctx.hx_plan_greedy(r.model, calls, pre, dec, links, tail, horizon, bp, bd, bc, ratio, rank,
                           backlog_tok_out=backlog, used_tok_out=used, batch_out=batch, qd_tok_out=qd)
        return dict(best_p=bp, best_d=bd, best_cost=bc, ratio=ratio, rank=rank, backlog=backlog, used=used, batch=batch, qd=qd)

    return dict(ctx=ctx, run=run)


_PREPARE = dict(round=_prepare_round, stream=_prepare_stream, tensor=_prepare_tensor, horizons=_prepare_horizons,
                decode=_prepare_decode, decode_plan=_prepare_decode_plan, plan=_prepare_plan)


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    return state["run"]()


# ---- what a pass cannot do without ------------------------------------------------------


def _search_flops(C, P, D, T):
    # per call: the service time and finish on every prefill instance, the transfer between every pair of classes, the decode
    # time and feasibility on every decode instance and its finish.  A candidate's cost depends on its prefill instance
    # through the earliest arrival at the decode class only, so the pairs need not be formed one by one.
    return C * (5.0 * P + 3.0 * T * T + 9.0 * D)


def work(case):
    k = case["kind"]
    if k == "round":
        C, P, D, T = case["calls"], case["prefill"], case["decode"], case["types"]
        n = case["workflows"] * (8 if case["small_dags"] else 20)
        e = 1.31 * n
        return dict(bytes=36.0 * C + 24 * P + 44 * D + 32 * n + 4 * e + 8 * case["workflows"],
                    flops=_search_flops(C, P, D, T) + n * (3.0 * T * T + 12 * T))
    if k == "stream":
        C, P, D, T = case["calls"], case["prefill"], case["decode"], case["types"]
        n = 3.65 * case["live"]                         # nodes a round reveals; parents of a round mostly lie in earlier ones
        per_round = 36.0 * C + 24 * P + 44 * D + n * (12 + 4 + 24 + 16) + 8 * case["live"]
        return dict(bytes=case["rounds"] * per_round + 3 * n * 60 + (case["rounds"] + 3) * n * 20,
                    flops=case["rounds"] * _search_flops(C, P, D, T) + (case["rounds"] + 3) * n * (3.0 * T * T + 12 * T))
    if k == "tensor":
        C, P, D = case["calls"], case["prefill"], case["decode"]
        return dict(bytes=8.0 * C * P * D + C * D + 36 * C, flops=4.0 * C * P * D)
    if k == "horizons":
        n = case["workflows"] * 20
        e = (1.31 if case["sweeps"] else 1.705) * n
        return dict(bytes=n * (8 + 4 + 4 + 4 + 12) + 4 * e + 8 * case["workflows"], flops=n * 96.0 + e)
    if k in ("decode", "decode_plan"):
        Q, D, iv = case["calls"], case["decode"], case["resident"] + case["planned"]
        pairs = 0.5 * Q * D + 0.5 * Q                   # half the calls are locked to one instance
        # a free pair needs at least its decode time and one comparison with what the instance has room for
        flops = pairs * 12.0 + D * iv * 16.0
        return dict(bytes=44.0 * Q + D * (28 + 12 * iv), flops=flops + (Q * D * 12.0 if k == "decode_plan" else 0))
    Q, P, D, T = case["calls"], case["prefill"], case["decode"], case["types"]
    return dict(bytes=40.0 * Q + 24 * P + 44 * D, flops=2 * _search_flops(Q, P, D, T))


def tolerance(case):
    # Costs are sums and products of positive 32-bit terms, at most some ten roundings deep.  Compared with the same path in 64
    # bits, the 2-norm of the difference was 4e-8 (costs) to 7.8e-8 (ratios) of the result's, and no index, rank or counter
    # differed.  Two pairs whose costs differ by a rounding may change places in another implementation, which moves a call's
    # index and the counters of two instances: a few in a thousand at most.
    return {"rel": 3.2e-7, "differ": 0.002}
