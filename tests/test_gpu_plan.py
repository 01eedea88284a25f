"""GPU parity of the planner around the scoring loop: one-pass ordering and the
recomputing greedy loop (Algorithm 1 main loop; Sec. 5.3), through the C ABI.

The greedy sequence is chaotic under fp32 near-ties (a different pick changes
every later state), so the plan is checked step by step: the oracle replays the
GPU's order on its own copy of the state, and at every step the GPU's call must
be a most-urgent one and its pair an earliest-finish one up to the fp32
tolerance; only then is it applied to the oracle's state.  Integer state must
agree exactly at the end."""
import numpy as np
import pytest

from oracle import hx_oracle as o
from paper_2605_16637_amd import synth
from gpu_helpers import REL, assert_costs_close, dev
from helpers import random_pool

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2605_16637_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("C", [1, 7, 2048, 2049, 16384, 16385, 40000, 100003])
def test_rank_matches_oracle(ctx, C):
    import torch
    rng = np.random.default_rng(60 + C)
    r = rng.choice(np.concatenate([rng.uniform(0.1, 5.0, 50), [np.inf, 2.0, 2.0]]), C).astype(np.float32)
    want = o.rank(r.astype(np.float64)) if C <= 2049 else None
    rank = torch.full((C,), -1, dtype=torch.int32, device="cuda:0")
    ctx.hx_rank(dev(r), rank)
    ctx.hx_stream_status()
    got = rank.cpu().numpy()
    if want is None:        # the quadratic oracle is too slow here: a stable sort gives the same definition
        order = np.argsort(-r.astype(np.float64), kind="stable")
        want = np.empty(C, np.int64); want[order] = np.arange(C)
    assert np.array_equal(got, want)


# the ordering where its tiles can go wrong: the sizes around their limits, all ratios equal, all infinite, ratios over
# many magnitudes and of either sign, a few values a rounding apart
@pytest.mark.parametrize("C", [63, 64, 65, 1025, 2048, 2049, 8192, 8193, 16384])
@pytest.mark.parametrize("kind", ["equal", "infinite", "magnitudes", "close"])
def test_rank_of_unusual_ratios(ctx, C, kind):
    import torch
    rng = np.random.default_rng(C)
    r = {"equal": np.full(C, 0.7), "infinite": np.full(C, np.inf),
         "magnitudes": 10.0 ** rng.uniform(-37, 37, C) * rng.choice([-1, 1], C),
         "close": np.float32(1.5) + rng.integers(0, 3, C) * np.finfo(np.float32).eps}[kind].astype(np.float32)
    if kind == "magnitudes":
        r[rng.integers(0, C, 5)] = [np.inf, -np.inf, 0.0, np.inf, np.float32(3.4e38)]
    rank = torch.full((C,), -1, dtype=torch.int32, device="cuda:0")
    ctx.hx_rank(dev(r), rank)
    ctx.hx_stream_status()
    order = np.argsort(-r.astype(np.float64), kind="stable")
    want = np.empty(C, np.int64); want[order] = np.arange(C)
    assert np.array_equal(rank.cpu().numpy(), want)


@pytest.mark.parametrize("C", [40, 1024, 3000, 20000])      # one launch, at most; all pairs; by buckets
def test_rank_puts_a_ratio_that_is_no_number_with_the_infinite(ctx, C):
    import torch
    rng = np.random.default_rng(C)
    r = rng.uniform(0.1, 5.0, C).astype(np.float32)
    odd = rng.choice(C, 9, replace=False)
    r[odd[:5]] = np.nan; r[odd[5:]] = np.inf
    rank = torch.full((C,), -1, dtype=torch.int32, device="cuda:0")
    ctx.hx_rank(dev(r), rank)
    ctx.hx_stream_status()
    order = np.argsort(-np.where(np.isnan(r), np.inf, r), kind="stable")
    want = np.empty(C, np.int64); want[order] = np.arange(C)
    assert np.array_equal(rank.cpu().numpy(), want)


# the lines between the ways of ordering (10240 and 28672 calls), and queues whose calls mostly fall between two of the
# calls that divide it: more in one bucket than a workgroup holds of it
@pytest.mark.parametrize("C", [10240, 10241, 28672, 28673])
@pytest.mark.parametrize("kind", ["spread", "sorted", "few values", "one bucket"])
def test_rank_between_cuts(ctx, C, kind):
    import torch
    rng = np.random.default_rng(C)
    r = rng.lognormal(0, 1, C)
    if kind == "sorted":
        r = np.sort(r)
    elif kind == "few values":
        r = rng.choice([0.5, 1.5, -2.0, np.inf, -np.inf], C)
    elif kind == "one bucket":
        # the call that each of 255 stretches gives as a divider is larger than all others
        t = np.arange(255, dtype=np.int64)
        begin = t * C // 256
        size = (t + 1) * C // 256 - begin
        hashed = (t * 2654435761 % 2 ** 32) >> 8
        r[begin + (hashed * size >> 24)] += 1e6
    r = r.astype(np.float32)
    rank = torch.full((C + 64,), -1, dtype=torch.int32, device="cuda:0")
    ctx.hx_rank(dev(r), rank[:C])
    ctx.hx_stream_status()
    order = np.argsort(-r.astype(np.float64), kind="stable")
    want = np.empty(C, np.int64); want[order] = np.arange(C)
    assert np.array_equal(rank[:C].cpu().numpy(), want) and bool((rank[C:] == -1).all())


# A queue whose dividers all lie above the other calls.  The workgroup that gets the bucket sorts it 4096 calls at a time and looks
# every call up in each part, some 92 us a part (7 of them at most) beside the 11 to 25 us of a queue that divides well: 15 to 26
# times that.  Counted pair by pair it was 600 to 2000 times.
@pytest.mark.parametrize("C", [10241, 16384, 28672])
def test_rank_time_of_one_bucket(ctx, C):
    import torch
    rng = np.random.default_rng(C)
    even = rng.random(C).astype(np.float32)
    t = np.arange(255, dtype=np.int64)
    begin = t * C // 256
    size = (t + 1) * C // 256 - begin
    uneven = even.copy()
    uneven[begin + ((t * 2654435761 % 2 ** 32 >> 8) * size >> 24)] += 2
    rank = torch.empty(C, dtype=torch.int32, device="cuda:0")
    times = []
    for r in (dev(even), dev(uneven)):
        run = ctx.prepare(lambda: ctx.hx_rank(r, rank))
        run()
        best = np.inf
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                run()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 4)
        times.append(best)
    assert times[1] < 100 * times[0], times


# members of one bucket around what a workgroup counts by pairs, what it sorts at once and what it sorts in parts: 0, 1 or some
# above all dividers, the others between the first two, below all or in one run
@pytest.mark.parametrize("n", [1, 63, 65, 255, 257, 575, 767, 768, 769, 1023, 1024, 1025, 2047, 2049, 4095, 4096, 4097, 8200])
@pytest.mark.parametrize("where", ["above", "between", "below"])
def test_rank_with_a_bucket_of(ctx, n, where):
    import torch
    C = 12000
    rng = np.random.default_rng(n)
    t = np.arange(255, dtype=np.int64)
    begin = t * C // 256
    size = (t + 1) * C // 256 - begin
    cut = begin + ((t * 2654435761 % 2 ** 32 >> 8) * size >> 24)
    # dividers at 1 .. 255; the n members between two of them (or at an end), some ratios among them equal; all other calls spread
    r = rng.uniform(1, 255, C)
    r[cut] = rng.permutation(np.arange(1, 256))
    members = rng.choice(np.setdiff1d(np.arange(C), cut), n, replace=False)
    r[members] = {"above": 300, "between": 100.25, "below": -5}[where] + rng.integers(0, max(2, n // 2), n) / (4 * n + 8)
    r = r.astype(np.float32)
    rank = torch.full((C + 64,), -1, dtype=torch.int32, device="cuda:0")
    ctx.hx_rank(dev(r), rank[:C])
    ctx.hx_stream_status()
    order = np.argsort(-r.astype(np.float64), kind="stable")
    want = np.empty(C, np.int64); want[order] = np.arange(C)
    assert np.array_equal(rank[:C].cpu().numpy(), want) and bool((rank[C:] == -1).all())


def run_greedy(ctx, model, L, O, elapsed, node, wf, tail, hor, pre, dec, links):
    import torch
    from paper_2605_16637_amd import binding
    C, P, D = len(L), len(pre["flops"]), len(dec["flops"])
    calls = binding.to_device(dict(n=C, L_in=np.asarray(L, np.int32), L_out=np.asarray(O, np.int32),
                                   node=np.asarray(node, np.int32), wf=np.asarray(wf, np.int32),
                                   elapsed=np.asarray(elapsed, np.float32)))
    dp = binding.to_device({**{k: np.asarray(v) for k, v in pre.items()}, "n": P})
    dd = binding.to_device({**{k: np.asarray(v) for k, v in dec.items()}, "n": D})
    dl = binding.to_device(links)
    i32 = dict(dtype=torch.int32, device="cuda:0")
    bp, bd, rk = torch.full((C,), -9, **i32), torch.full((C,), -9, **i32), torch.full((C,), -9, **i32)
    bc, rt = torch.full((C,), -9.0, device="cuda:0"), torch.full((C,), -9.0, device="cuda:0")
    st = [torch.full((P,), -9, **i32)] + [torch.full((D,), -9, **i32) for _ in range(3)]
    ctx.hx_plan_greedy(model, calls, dp, dd, dl, dev(np.asarray(tail, np.float32)), dev(np.asarray(hor, np.float32)),
                       bp, bd, bc, rt, rk, *st)
    ctx.hx_stream_status()
    return [x.cpu().numpy() for x in (bp, bd, bc, rt, rk, *st)]


def check_plan_stepwise(model, L, O, elapsed, node, wf, tail, hor, pre, dec, links, got):
    gp, gd, gc, gr, grank, g_bl, g_us, g_ba, g_qd = got
    C = len(L)
    assert sorted(grank) == list(range(C))
    sp = {k: np.array(v).copy() for k, v in pre.items()}
    sd = {k: np.array(v).copy() for k, v in dec.items()}
    alive = list(range(C))
    elapsed = np.asarray(elapsed, np.float32).astype(np.float64)
    tail = np.asarray(tail, np.float32).astype(np.float64); hor = np.asarray(hor, np.float32).astype(np.float64)
    L, O = np.asarray(L), np.asarray(O)
    for k in range(C):
        c = int(np.nonzero(grank == k)[0][0])
        s = o.score(model, L[alive], O[alive], sp, sd, links)
        with np.errstate(all="ignore"):
            R = (elapsed[alive] + s.best_cost + tail[np.asarray(node)[alive]]) / hor[np.asarray(wf)[alive]]
        i = alive.index(c)
        # the picked call is a most urgent one (exactly, or within the fp32 tolerance of the largest ratio)
        top = R.max()
        assert (np.isinf(top) and np.isinf(R[i])) or R[i] >= top * (1 - 2 * REL), f"step {k}: call {c} ratio {R[i]} vs {top}"
        if np.isinf(R[i]):
            assert (gp[c], gd[c]) == (-1, -1) and np.isinf(gc[c]) and np.isinf(gr[c])
            # among calls with nothing feasible the lowest index goes first
            assert c == min(a for a, r in zip(alive, R) if np.isinf(r))
        else:
            assert gp[c] >= 0 and gd[c] >= 0
            alt = o.score_one(model, L[c], O[c], gp[c], gd[c], sp, sd, links)
            assert np.isfinite(alt) and alt <= s.best_cost[i] * (1 + REL), f"step {k}: pair of call {c}"
            assert abs(gc[c] - alt) <= REL * alt
            want_r = (elapsed[c] + alt + tail[node[c]]) / hor[wf[c]]
            assert abs(gr[c] - want_r) <= REL * want_r
            p, d = int(gp[c]), int(gd[c])
            sp["backlog_tok"][p] += L[c]
            sd["qd_tok"][d] += O[c]; sd["used_tok"][d] += L[c] + O[c]
            sd["batch"][d] = min(256, -(-int(sd["used_tok"][d]) // 2048))
        alive.remove(c)
    assert np.array_equal(g_bl, sp["backlog_tok"]) and np.array_equal(g_us, sd["used_tok"])
    assert np.array_equal(g_ba, sd["batch"]) and np.array_equal(g_qd, sd["qd_tok"])


@pytest.mark.parametrize("C,P,D,T,seed", [(3, 2, 2, 2, 1), (24, 8, 8, 3, 2), (64, 8, 10, 3, 3), (40, 64, 64, 4, 4),
                                          (130, 20, 33, 8, 5), (16, 256, 256, 8, 6),
                                          # the queue and pool bench.py times
                                          (256, 64, 64, 4, 7),
                                          # pools searched class by class (more than 64 x 64 pairs)
                                          (60, 100, 90, 5, 8), (48, 70, 256, 3, 9)])
def test_greedy_plan_matches_oracle(ctx, C, P, D, T, seed):
    rng = np.random.default_rng(70 + seed)
    model = synth.MODEL
    types, pre, dec, links = random_pool(rng, P, D, T)
    # tight capacities: calls stop fitting as the plan fills the pool
    dec["cap_tok"] = (dec["used_tok"] + rng.integers(2000, 60000, D)).astype(np.int32)
    L, O = synth.gen_lengths(rng, C)
    elapsed = rng.uniform(0, 20, C).astype(np.float32)
    n_nodes, n_wf = C + 5, 4
    node = rng.permutation(n_nodes)[:C].astype(np.int32); wf = rng.integers(0, n_wf, C).astype(np.int32)
    tail = rng.uniform(0, 5, n_nodes).astype(np.float32); hor = rng.uniform(5, 50, n_wf).astype(np.float32)
    got = run_greedy(ctx, model, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
    check_plan_stepwise(model, L, O, elapsed, node, wf, tail, hor, pre, dec, links, got)
    # and, when no near-tie occurred, the oracle's own plan is the same plan
    want = o.plan_greedy(model, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
    if np.array_equal(got[4], want.rank):
        assert np.array_equal(got[0], want.best_p) and np.array_equal(got[1], want.best_d)
        assert_costs_close(got[2], want.best_cost, "plan cost"); assert_costs_close(got[3], want.ratio, "plan ratio")
        assert np.array_equal(got[5], want.backlog_tok) and np.array_equal(got[6], want.used_tok)


# one call a lane up to the widest workgroup, the stages in which the remaining calls are dealt to the lanes anew, more than
# 64 instances of one side, more than four classes, groups of four decode instances that are not full, and prefill
# instances of one class with rates of their own (several entries of the search per class)
@pytest.mark.parametrize("C,P,D,T,seed", [(1, 1, 1, 1, 1), (65, 3, 5, 5, 2), (257, 9, 66, 3, 3), (90, 65, 7, 8, 4), (513, 5, 6, 2, 5)])
def test_greedy_plan_with_rates_of_every_instance(ctx, C, P, D, T, seed):
    rng = np.random.default_rng(170 + seed)
    types, pre, dec, links = random_pool(rng, P, D, T)
    for side, n in ((pre, P), (dec, D)):
        for k in ("flops", "hbm_bw"):
            # a third of the instances keep the rates of their class
            side[k] = (side[k] * np.where(rng.random(n) < 0.33, 1.0, rng.uniform(0.7, 1.4, n))).astype(np.float32)
    dec["cap_tok"] = (dec["used_tok"] + rng.integers(2000, 90000, D)).astype(np.int32)
    L, O = synth.gen_lengths(rng, C)
    elapsed = rng.uniform(0, 20, C).astype(np.float32)
    node = rng.permutation(C).astype(np.int32); wf = rng.integers(0, 3, C).astype(np.int32)
    tail = rng.uniform(0, 5, C).astype(np.float32); hor = rng.uniform(5, 50, 3).astype(np.float32)
    got = run_greedy(ctx, synth.MODEL, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
    check_plan_stepwise(synth.MODEL, L, O, elapsed, node, wf, tail, hor, pre, dec, links, got)


# the batch after each pick is a division by tokens_per_seq, the availability hint one by the nominal batch (a
# multiplication where that is a power of two)
@pytest.mark.parametrize("tokens_per_seq", [1, 3, 2047, 4096, 2 ** 31 - 1])
@pytest.mark.parametrize("bbar", [48.0, 0.25])
def test_greedy_plan_divides_exactly(ctx, tokens_per_seq, bbar):
    import torch
    from paper_2605_16637_amd import binding
    rng = np.random.default_rng(tokens_per_seq % 1000)
    C, P, D, model = 40, 5, 9, dict(synth.MODEL, nominal_batch=bbar)
    types, pre, dec, links = random_pool(rng, P, D, 3)
    dec["cap_tok"] = (dec["used_tok"] + rng.integers(2000, 2 ** 28, D)).astype(np.int32)
    L, O = synth.gen_lengths(rng, C)
    elapsed = rng.uniform(0, 20, C).astype(np.float32)
    node, wf = np.arange(C, dtype=np.int32), rng.integers(0, 3, C).astype(np.int32)
    tail = rng.uniform(0, 5, C).astype(np.float32); hor = rng.uniform(5, 50, 3).astype(np.float32)
    if tokens_per_seq == 4096:                  # the whole plan, with the method's own rule
        got = run_greedy(ctx, model, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
        check_plan_stepwise(model, L, O, elapsed, node, wf, tail, hor, pre, dec, links, got)
    calls = binding.to_device(dict(n=C, L_in=L, L_out=O, node=node, wf=wf, elapsed=elapsed))
    dp, dd = (binding.to_device({**{k: np.asarray(v) for k, v in t.items()}, "n": n}) for t, n in ((pre, P), (dec, D)))
    out = [torch.empty(n, dtype=t, device="cuda:0") for n, t in ((C, torch.int32), (C, torch.int32), (C, torch.float32), (C, torch.float32),
                                                                 (C, torch.int32), (P, torch.int32), (D, torch.int32), (D, torch.int32), (D, torch.int32))]
    ctx.hx_plan_greedy(model, calls, dp, dd, binding.to_device(links), dev(tail), dev(hor), *out, tokens_per_seq=tokens_per_seq,
                       max_batch=10 ** 6)
    ctx.hx_stream_status()
    used, batch = out[6].cpu().numpy().astype(np.int64), out[7].cpu().numpy()
    took = np.isin(np.arange(D), out[1].cpu().numpy())
    assert took.any()
    assert np.array_equal(batch, np.where(took, np.minimum(-(-used // tokens_per_seq), 10 ** 6), dec["batch"]))


# Plans that begin with more decode times than the workgroup's memory keeps and end with few enough: up to 512 calls with small
# and large pools, and more
@pytest.mark.parametrize("C,P,D,T,seed", [(512, 8, 64, 8, 1), (400, 66, 90, 4, 2), (1024, 4, 18, 3, 3)])
def test_greedy_plan_whose_decode_times_are_not_kept_at_first(ctx, C, P, D, T, seed):
    rng = np.random.default_rng(270 + seed)
    types, pre, dec, links = random_pool(rng, P, D, T)
    groups = int(sum(-(-int((dec["type"] == t).sum()) // 4) for t in range(T)))
    assert ctx.lib.hx_test_plan_stages(C, D, T, groups) == 3              # some stages keep them, some do not
    dec["cap_tok"] = (dec["used_tok"] + rng.integers(20000, 300000, D)).astype(np.int32)
    L, O = synth.gen_lengths(rng, C)
    elapsed = rng.uniform(0, 20, C).astype(np.float32)
    node = rng.permutation(C).astype(np.int32); wf = rng.integers(0, 3, C).astype(np.int32)
    tail = rng.uniform(0, 5, C).astype(np.float32); hor = rng.uniform(5, 50, 3).astype(np.float32)
    got = run_greedy(ctx, synth.MODEL, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
    check_plan_stepwise(synth.MODEL, L, O, elapsed, node, wf, tail, hor, pre, dec, links, got)
    assert (got[0] >= 0).sum() > C // 2


def test_greedy_hand_worked_conflict_on_gpu(ctx):
    from helpers import ROUND_MODEL, read_kv
    G = read_kv("round_numbers.txt")
    pre = dict(flops=np.array([1e13, 1e13], np.float32), hbm_bw=np.array([1e12, 1e12], np.float32),
               backlog_tok=np.zeros(2, np.int32), type=np.zeros(2, np.int32))
    dec = dict(flops=np.array([1e13], np.float32), hbm_bw=np.array([1e12], np.float32), used_tok=np.zeros(1, np.int32),
               cap_tok=np.array([10**6], np.int32), batch=np.zeros(1, np.int32), qd_tok=np.zeros(1, np.int32),
               type=np.zeros(1, np.int32))
    links = dict(n_types=1, bw=np.array([[1e9]], np.float32), latency=np.array([[0.05]], np.float32))
    gp, gd, gc, gr, grank, bl, us, ba, qd = run_greedy(ctx, ROUND_MODEL, [1000, 1000], [100, 100], [1.0, 5.0], [0, 1], [0, 0],
                                                        [0.0, 0.0], [10.0], pre, dec, links)
    assert list(grank) == [1, 0] and list(gp) == [1, 0] and list(gd) == [0, 0]
    assert gc[1] == pytest.approx(G["greedy_A_cost"], rel=REL) and gc[0] == pytest.approx(G["greedy_B_cost"], rel=REL)
    assert gr[1] == pytest.approx(G["greedy_A_ratio"], rel=REL) and gr[0] == pytest.approx(G["greedy_B_ratio"], rel=REL)
    assert list(bl) == [1000, 1000] and list(us) == [2200] and list(qd) == [200] and list(ba) == [2]


@pytest.mark.parametrize("P,D", [(6, 5), (96, 80)])
def test_greedy_breaks_exact_ties_by_lowest_index(ctx, P, D):
    # identical instances on both sides (two classes, all of a class in the same state): every call sees exact ties
    # over many pairs; the plan has to be the oracle's pair for pair, the lowest (p, d) among equals at every step --
    # on a small pool (searched pair by pair) and on a large one (searched class by class)
    rng = np.random.default_rng(P)
    C = 40
    tp, td = (np.arange(P) % 2).astype(np.int32), (np.arange(D) % 2).astype(np.int32)
    F, B = np.array([4e14, 1e15], np.float32), np.array([2e12, 3.3e12], np.float32)
    pre = dict(flops=F[tp], hbm_bw=B[tp], backlog_tok=np.zeros(P, np.int32), type=tp)
    dec = dict(flops=F[td], hbm_bw=B[td], used_tok=np.full(D, 4096, np.int32), cap_tok=np.full(D, 10**6, np.int32),
               batch=np.full(D, 2, np.int32), qd_tok=np.zeros(D, np.int32), type=td)
    links = dict(n_types=2, bw=np.array([[5e10, 2.5e10], [2.5e10, 1e11]], np.float32), latency=np.zeros((2, 2), np.float32))
    L, O = synth.gen_lengths(rng, C)
    elapsed = rng.uniform(0, 20, C).astype(np.float32)
    node = np.arange(C, dtype=np.int32); wf = (np.arange(C) % 4).astype(np.int32)
    tail = rng.uniform(0, 5, C).astype(np.float32); hor = rng.uniform(5, 50, 4).astype(np.float32)
    got = run_greedy(ctx, synth.MODEL, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
    want = o.plan_greedy(synth.MODEL, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
    assert np.array_equal(got[4], want.rank)
    assert np.array_equal(got[0], want.best_p) and np.array_equal(got[1], want.best_d)
    assert_costs_close(got[2], want.best_cost, "plan cost")
    # the first call placed had the whole pool to choose from, all instances of a class equal: it took the first of its classes
    first = int(np.argmin(got[4]))
    assert got[0][first] < 2 and got[1][first] < 2


def test_planner_limits_and_empty_inputs(ctx):
    import torch
    from paper_2605_16637_amd import binding
    rng = np.random.default_rng(80)
    types, pre, dec, links = random_pool(rng, 4, 4, 2)
    L, O = synth.gen_lengths(rng, 5)
    # an empty decode pool: nothing is feasible, calls are ranked by index, the state comes back unchanged
    none = {k: np.asarray(v)[:0] for k, v in dec.items()}
    got = run_greedy(ctx, synth.MODEL, L, O, np.ones(5), np.arange(5), np.zeros(5, int), np.zeros(5), [9.0], pre, none, links)
    assert (got[0] == -1).all() and np.isinf(got[2]).all() and list(got[4]) == [0, 1, 2, 3, 4]
    assert np.array_equal(got[5], pre["backlog_tok"])
    # beyond the queue length the planner takes
    C = 1025
    big = binding.to_device(dict(n=C, L_in=np.ones(C, np.int32), L_out=np.ones(C, np.int32), node=np.zeros(C, np.int32),
                                 wf=np.zeros(C, np.int32), elapsed=np.zeros(C, np.float32)))
    i32 = dict(dtype=torch.int32, device="cuda:0")
    out = [torch.empty(C, **i32), torch.empty(C, **i32), torch.empty(C, device="cuda:0"), torch.empty(C, device="cuda:0"),
           torch.empty(C, **i32)]
    pre["n"], dec["n"] = 4, 4
    with pytest.raises(binding.HxError) as e:
        ctx.hx_plan_greedy(synth.MODEL, big, binding.to_device(pre), binding.to_device(dec), binding.to_device(links),
                           dev(np.zeros(1, np.float32)), dev(np.ones(1, np.float32)), *out)
    assert e.value.code == -2


def test_greedy_rescans_everything_when_a_commit_lowers_a_term(ctx):
    # The snapshot's batch of a decode instance may stand above what the batch rule gives for its occupancy (the
    # interface only asks for batch >= 0).  The first commit on that instance then lowers its per-token time, pairs
    # on it get cheaper, and calls whose current pair is elsewhere must move there: the plan is Algorithm 1's full
    # recomputation only if those calls are scored again.  Compute-bound decode (large FLOP per token) makes the
    # batch term the one that counts; two decode classes, the fast instance starting with the inflated batch.
    rng = np.random.default_rng(91)
    model = dict(synth.MODEL); model["flops_per_token"] = 4e11
    P, D, C = 6, 2, 24
    tp = (np.arange(P) % 2).astype(np.int32); td = np.array([1, 0], np.int32)
    F, B = np.array([4e14, 1e15], np.float32), np.array([2e12, 3.3e12], np.float32)
    pre = dict(flops=F[tp], hbm_bw=B[tp], backlog_tok=rng.integers(0, 3000, P).astype(np.int32), type=tp)
    L, O = synth.gen_lengths(rng, C)
    dec = dict(flops=F[td], hbm_bw=B[td], used_tok=np.array([20000, 20000], np.int32),
               cap_tok=np.array([10**6, 20000 + int(np.median(L + O)) * 6], np.int32),
               batch=np.array([150, 12], np.int32), qd_tok=np.array([500, 500], np.int32), type=td)
    links = dict(n_types=2, bw=np.array([[5e10, 2.5e10], [2.5e10, 1e11]], np.float32), latency=np.zeros((2, 2), np.float32))
    elapsed = rng.uniform(0, 20, C).astype(np.float32)
    node = np.arange(C, dtype=np.int32); wf = (np.arange(C) % 4).astype(np.int32)
    tail = rng.uniform(0, 5, C).astype(np.float32); hor = rng.uniform(5, 50, 4).astype(np.float32)
    want = o.plan_greedy(model, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
    # the case is what it is meant to be: on the snapshot every call prefers instance 1; once a call has gone to
    # instance 0 its batch falls from 150 and most of the remaining calls follow
    snap = o.score(model, L, O, pre, dec, links)
    assert (snap.best_d == 1).all() and want.batch[0] < 150 and (want.best_d == 0).sum() > C // 2
    got = run_greedy(ctx, model, L, O, elapsed, node, wf, tail, hor, pre, dec, links)
    check_plan_stepwise(model, L, O, elapsed, node, wf, tail, hor, pre, dec, links, got)
    assert np.array_equal(got[4], want.rank)
    assert np.array_equal(got[0], want.best_p) and np.array_equal(got[1], want.best_d)
    assert_costs_close(got[2], want.best_cost, "plan cost")
    assert np.array_equal(got[7], want.batch) and np.array_equal(got[6], want.used_tok)
