// Workflow horizons: standalone node cost, the max-plus critical-path pass
// (single-pass workflow-local form and level-synchronous general form) and the
// incremental append for DAGs revealed at run time.
//
// What is computed: Sec. 5.1 of the paper.  H_w(t) is the completion time of
// the revealed sub-DAG of workflow w served in isolation; it is recomputed when
// calls are revealed and can only grow.  Here that is the longest
// cost-weighted path, with rem[v] = cost[v] + max over successors of rem.
//
// rem is one fp32 addition of an exact maximum, so every evaluation order --
// the single pass, the sweeps, the incremental propagation -- gives the same
// bits.
#include "hx_common.hpp"
#include "hx_terms.hpp"
#include "hx_search.hpp"
#include "hx_cp.hpp"
#include "hx_append.hpp"

#include <cmath>

namespace {

// ---- standalone node cost -----------------------------------------------------

// NN nodes a thread at a time, 256 apart, so that every load is coalesced and NN of each kind are in flight.  AT_ONCE: all pairs of
// classes at once.
template <int NN, int TT, bool AT_ONCE = false>
__global__ __launch_bounds__(256) void hx_node_cost_kernel(NodeCostArgs a)
{
    __shared__ CostTables s_tab;
    const int tid = threadIdx.x;
    int L[NN], O[NN];
    float c[NN];
    // the first nodes' lengths are on their way while the class tables are set up
    auto load = [&](int v0) {
#pragma unroll
        for (int n = 0; n < NN; ++n) {
            const int v = (int)min((unsigned)v0 + n * 256u, (unsigned)a.n - 1u);
            L[n] = a.L_in[v]; O[n] = a.L_out[v];
        }
    };
    const long long step = (long long)gridDim.x * (256 * NN);
    long long at = (long long)blockIdx.x * (256 * NN) + tid;
    load((int)min(at, (long long)a.n - 1));
    hx_cost_tables_fill(s_tab, a, tid);
    __syncthreads();
    for (; at < a.n; at += step) {
        if constexpr (AT_ONCE) c[0] = hx_node_cost_at_once(a.m, s_tab, a.T, L[0], O[0]);
        else hx_node_cost_eval<NN, TT>(a.m, s_tab, a.T, L, O, c);
#pragma unroll
        for (int n = 0; n < NN; ++n)
            if (at + n * 256 < a.n) a.cost[at + n * 256] = c[n];
        if (at + step < a.n) load((int)(at + step));
    }
}


// ---- critical path, single pass ---------------------------------------------------

template <bool STREAM>
__global__ __launch_bounds__(CP_THREADS) __attribute__((amdgpu_waves_per_eu(7, 8)))
void hx_cp_local_kernel(CpArgs a, int wpb)
{
    __shared__ CpNode s_node[CP_NMAX + 1];
    __shared__ int s_any;                     // == first workflow of the run + 1: a node of this run was left to the walk
    hx_cp_local_body<CP_NMAX, false, STREAM>(a, wpb, s_node, s_any, nullptr, nullptr, (int)blockIdx.x);
}

// The same pass with the standalone node cost worked out while staging instead of being read:
// one launch for what hx_node_cost_kernel and hx_cp_local_kernel do one after the other.  The
// staging with the cost's sums in flight takes 102 registers, four wavefronts a SIMD; the launch is
// meant for the graphs of a scheduling round (tens of thousands of nodes, spread over all compute
// units), where the latency of a launch counts and residency does not.
// WAVES: `wpv` workflows to a wavefront where all of a workgroup's are small enough (hx_cp_wave); else the workgroup
// takes its `wpb` = 4 * wpv workflows, which may be more than CP_WPB, in runs of at most that many.
template <bool WAVES>
__global__ __launch_bounds__(CP_THREADS)
void hx_cp_cost_kernel(CpArgs a, NodeCostArgs nc, int wpb, int wpv)
{
    __shared__ union {
        CpNode node[CP_NMAX_COST + 1];
        CpWave wave[CP_THREADS / HX_WAVE];
    } s;
    __shared__ int s_any;
    __shared__ CostTables s_tab;
    if constexpr (WAVES)
        if (hx_cp_waves_body<CP_THREADS>(a, wpb, wpv, s.wave, nc, s_tab, (int)blockIdx.x)) return;
    hx_cp_local_body<CP_NMAX_COST, true, false>(a, wpb, s.node, s_any, &nc, &s_tab, (int)blockIdx.x, WAVES);
}

// ---- critical path, level-synchronous sweeps ------------------------------------------
//
// Successors may be anywhere, but in nearly every graph they lie in their node's workflow, or near it.  A workgroup takes a
// slice of whole workflows into LDS and sweeps there, a barrier a sweep, until nothing changes.  Where that does not
// finish the graph a second kernel sweeps it as a whole, from the values the slices left if only edges between them (or
// malformed rows) are missing, from the beginning if some nodes have no value yet (a workflow that does not fit, nodes of
// no workflow) or a slice was still changing at the limit (a cycle, or too small a limit).  Values only grow, towards
// the one fixed point there is, so both ways and every order give the same bits.
// Against a launch a sweep, 14 sweeps allowed: 20000 nodes in 1000 workflows of depth 12 64 -> 21 us, 1.8 million in
// 90000 276 -> 42; with one edge into another slice 64 -> 26 (20000 nodes) and 96 -> 36 (400000); every successor
// anywhere in the graph 79 -> 71 and 173 -> 177.
constexpr int CS_THREADS = 256;
constexpr int CS_NMAX = 1024;         // nodes of a slice
constexpr int CS_NPT = CS_NMAX / CS_THREADS;

// words of the context's d_sync, all 0 between launches; the counter of arrivals and the word that is polled have cache
// lines of their own (polls would hold the arrivals up)
enum : int { SY_AGAIN = 0, SY_OVER = 1, SY_LEFT = 2, SY_STUCK = 3, SY_COUNT = 32, SY_GO = 64 };
static_assert(SY_GO + 2 == HX_SYNC_WORDS, "two words each for the last two");

// WAVES: `wpv` workflows to a wavefront where all of a workgroup's are small enough (hx_cp_wave); an edge between two
// wavefronts' workflows is then one that the second kernel follows.
template <bool WAVES>
__global__ __launch_bounds__(CS_THREADS) void hx_cp_sweep_slices_kernel(CpArgs a, int wpb, int wpv, int max_sweeps, int32_t *sync)
{
    __shared__ union {
        int2 val[CS_NMAX + 1];                             // (rem, level) of node n0 + i at i + 1; 0: the empty successor
        CpWave wave[CS_THREADS / HX_WAVE];
    } s_lds;
    int2 *const s_val = s_lds.val;
    __shared__ int s_changed[3];
    const int tid = threadIdx.x;
    int w1 = min(((int)blockIdx.x + 1) * wpb, a.n_wf);
    bool odd = false, over = false;                        // over: not every node has been given a value
    if constexpr (WAVES) {
        const int lane = tid & (HX_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int wa = min((int)blockIdx.x * wpb + wave * wpv, a.n_wf), wb = min(wa + wpv, a.n_wf);
        const int p = hx_cp_wave_bounds(a, wa, wb, lane);
        if (!__syncthreads_or(hx_cp_wave_odd(a, p, wb - wa, lane))) {
            const CwFound f = hx_cp_wave<false, true>(a, wa, wb, p, s_lds.wave[wave], max_sweeps, nullptr, nullptr, lane);
            odd = f.not_dag || f.bad_index; over = f.over;
            w1 = 0;                                        // (no slice)
        }
    }
    if (w1 && tid == 0) s_val[0] = make_int2(0, -1);
    // nodes that belong to no workflow are swept too
    if (blockIdx.x == 0) over = over || a.wf_ptr[0] != 0 || a.wf_ptr[a.n_wf] != a.n_nodes;
    for (int wa = (int)blockIdx.x * wpb; wa < w1;) {
        // the run [wa, wb): as many of the slice's workflows as fit
        int wb = w1;
        const int n0 = a.wf_ptr[wa];
        int n1 = a.wf_ptr[wb];
        if (n0 < 0 || n1 < n0 || n1 > a.n_nodes) { over = true; break; }
        if (n1 - n0 > CS_NMAX) {
            int lo = wa, hi = wb;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                const int x = a.wf_ptr[mid];
                if (x >= n0 && x - n0 <= CS_NMAX) lo = mid; else hi = mid;
            }
            wb = max(lo, wa + 1);
            n1 = a.wf_ptr[wb];
            if (n1 < n0 || n1 > a.n_nodes || n1 - n0 > CS_NMAX) { over = true; break; }
        }
        const int nn = n1 - n0;
        float c[CS_NPT];
        int ra[CS_NPT], rb[CS_NPT], slot[CS_NPT][CP_DEG], tail[CS_NPT], lvl[CS_NPT];
        bool left[CS_NPT];                                 // more successors than slots, or a row at the very end of the id array
#pragma unroll
        for (int k = 0; k < CS_NPT; ++k) {
            const int v = n0 + min(k * CS_THREADS + tid, max(nn - 1, 0));
            const bool in = k * CS_THREADS + tid < nn;
            c[k] = in ? a.cost[v] : 0.0f;
            ra[k] = in ? a.row_ptr[v] : 0; rb[k] = in ? a.row_ptr[v + 1] : 0;
        }
#pragma unroll
        for (int k = 0; k < CS_NPT; ++k) {
            if (ra[k] < 0 || rb[k] > a.n_edges || ra[k] > rb[k]) { odd = true; ra[k] = rb[k] = 0; }
            const int deg = rb[k] - ra[k];
            left[k] = deg > CP_DEG || (deg > 0 && ra[k] > a.n_edges - CP_DEG);
            int id[CP_DEG] = {0, 0, 0, 0};
            if (a.n_edges >= CP_DEG) __builtin_memcpy(id, a.col + min(ra[k], a.n_edges - CP_DEG), sizeof id);
#pragma unroll
            for (int j = 0; j < CP_DEG; ++j) {
                const bool own = !left[k] && j < deg, here = (unsigned)(id[j] - n0) < (unsigned)nn;
                slot[k][j] = own && here ? id[j] - n0 + 1 : 0;
                odd = odd || (own && !here);
            }
            if (left[k]) for (int e = ra[k]; e < rb[k]; ++e) odd = odd || (unsigned)(a.col[e] - n0) >= (unsigned)nn;
            tail[k] = 0; lvl[k] = 0;
            if (k * CS_THREADS + tid < nn) s_val[k * CS_THREADS + tid + 1] = make_int2(__float_as_int(c[k]), 0);
        }
        if (tid < 3) s_changed[tid] = 0;
        __syncthreads();
        // Values another wavefront writes meanwhile may or may not be seen: they only grow, and a sweep in which nothing
        // was written has read final values.
        const int limit = min(max_sweeps, nn + 1);         // (only a cycle takes more than nn + 1)
        int s = 1;
        for (; s <= limit; ++s) {
            bool changed = false;
#pragma unroll
            for (int k = 0; k < CS_NPT; ++k) {
                if (k * CS_THREADS + tid >= nn) continue;
                const int2 g0 = s_val[slot[k][0]], g1 = s_val[slot[k][1]], g2 = s_val[slot[k][2]], g3 = s_val[slot[k][3]];
                // maxima of fp32 values that are not NaN with 0: those of their bits as signed integers
                int tb = max(max(max(g0.x, g1.x), max(g2.x, g3.x)), 0);
                int lv = max(max(g0.y, g1.y), max(g2.y, g3.y)) + 1;
                if (left[k]) for (int e = ra[k]; e < rb[k]; ++e) {
                    const unsigned i = (unsigned)(a.col[e] - n0);
                    if (i < (unsigned)nn) { const int2 g = s_val[i + 1]; tb = max(tb, g.x); lv = max(lv, g.y + 1); }
                }
                if (tb != tail[k] || lv != lvl[k]) {
                    changed = true;
                    tail[k] = tb; lvl[k] = lv;
                    s_val[k * CS_THREADS + tid + 1] = make_int2(__float_as_int(c[k] + __int_as_float(tb)), lv);
                }
            }
            if (changed) s_changed[s % 3] = 1;
            if (tid == 0) s_changed[(s + 1) % 3] = 0;
            __syncthreads();
            if (s_changed[s % 3] == 0) break;
        }
        if (s > limit) over = true;                        // still changing: a cycle, or the limit is too small
#pragma unroll
        for (int k = 0; k < CS_NPT; ++k) {
            const int i = k * CS_THREADS + tid;
            if (i < nn) {
                a.rem[n0 + i] = __int_as_float(s_val[i + 1].x); a.tail[n0 + i] = __int_as_float(tail[k]); a.level[n0 + i] = lvl[k];
            }
        }
        for (int w = wa + tid; w < wb; w += CS_THREADS) {
            const int ws = a.wf_ptr[w], we = a.wf_ptr[w + 1];
            if (ws < n0 || we > n1 || ws > we) { odd = true; continue; }
            int h = 0;
#pragma unroll 4
            for (int v = ws; v < we; ++v) h = max(h, s_val[v - n0 + 1].x);
            a.horizon[w] = __int_as_float(h);
        }
        __syncthreads();                                   // the next run stages over these values
        wa = wb;
    }
    // one store a workgroup (one a wavefront: 130 us with 590 workgroups)
    over = __syncthreads_or(over);
    odd = __syncthreads_or(odd);
    if (tid == 0 && over) sync[SY_OVER] = 1;
    if (tid == 0 && (over || odd)) sync[SY_AGAIN] = 1;
}

// Grid-wide sweeps: every node pulls from its successors.  What bounds them is latency, a chain of memory round trips a sweep:
// a thread takes CG_NPT nodes together, a step between them, and keeps their rows, successors and values in registers
// from sweep to sweep where that covers the graph, so that a sweep is the successors' values and no more.
constexpr int CG_THREADS = 512;
constexpr int CG_NPT = 4;

struct CgNodes {
    float c[CG_NPT], tail[CG_NPT];
    int lvl[CG_NPT], ra[CG_NPT], rb[CG_NPT], id[CG_NPT][CP_DEG];      // id: -1 where there is no successor
    bool left[CG_NPT];                                  // more successors than places, or a row at the very end of the id array
};

// the nodes v0, v0 + step, ..: rows and successors; tail and level as they were stored, or 0 (fresh)
__device__ __forceinline__ void hx_cp_nodes_load(const CpArgs &a, CgNodes &q, int v0, int step, bool fresh)
{
    bool bad = false;
#pragma unroll
    for (int k = 0; k < CG_NPT; ++k) {
        const long long at = v0 + (long long)k * step;
        const bool in = at < a.n_nodes;
        const int v = in ? (int)at : 0;
        q.c[k] = in ? a.cost[v] : 0.0f;
        q.ra[k] = in ? a.row_ptr[v] : 0; q.rb[k] = in ? a.row_ptr[v + 1] : 0;
        q.tail[k] = in && !fresh ? __hip_atomic_load(&a.tail[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0f;
        q.lvl[k] = in && !fresh ? __hip_atomic_load(&a.level[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    }
#pragma unroll
    for (int k = 0; k < CG_NPT; ++k) {
        if (q.ra[k] < 0 || q.rb[k] > a.n_edges || q.ra[k] > q.rb[k]) { bad = true; q.ra[k] = q.rb[k] = 0; }
        const int deg = q.rb[k] - q.ra[k];
        q.left[k] = deg > CP_DEG || (deg > 0 && q.ra[k] > a.n_edges - CP_DEG);
        int id[CP_DEG] = {0, 0, 0, 0};
        if (a.n_edges >= CP_DEG) __builtin_memcpy(id, a.col + min(q.ra[k], a.n_edges - CP_DEG), sizeof id);
#pragma unroll
        for (int j = 0; j < CP_DEG; ++j) {
            const bool own = !q.left[k] && j < deg, fine = (unsigned)id[j] < (unsigned)a.n_nodes;
            bad = bad || (own && !fine);
            q.id[k][j] = own && fine ? id[j] : -1;
        }
    }
    if (bad) hx_raise(a.status, HX_ERR_INDEX);
}

// One sweep over those nodes.  All that is written, and all that is read of what another thread writes, goes by device-scope
// atomics (also what no other workgroup reads in passing: nothing may lie in an XCD's cache when the last one redoes it).
__device__ __forceinline__ bool hx_cp_nodes_sweep(const CpArgs &a, CgNodes &q, int v0, int step)
{
    bool changed = false, bad = false;
    float r[CG_NPT][CP_DEG];
    int l[CG_NPT][CP_DEG];
#pragma unroll
    for (int k = 0; k < CG_NPT; ++k) {
#pragma unroll
        for (int j = 0; j < CP_DEG; ++j) {
            const int u = q.id[k][j];
            r[k][j] = 0.0f; l[k][j] = -1;
            if (u >= 0) {
                r[k][j] = __hip_atomic_load(&a.rem[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                l[k][j] = __hip_atomic_load(&a.level[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < CG_NPT; ++k) {
        float tl = fmaxf(fmaxf(fmaxf(r[k][0], r[k][1]), fmaxf(r[k][2], r[k][3])), 0.0f);
        int lv = max(max(l[k][0], l[k][1]), max(l[k][2], l[k][3])) + 1;
        if (q.left[k]) for (int e = q.ra[k]; e < q.rb[k]; ++e) {
            const int u = a.col[e];
            if (u < 0 || u >= a.n_nodes) { bad = true; continue; }
            tl = fmaxf(tl, __hip_atomic_load(&a.rem[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            lv = max(lv, __hip_atomic_load(&a.level[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1);
        }
        lv = min(lv, a.n_nodes);                        // a level beyond the node count can only come from a cycle: stop growing
        if (tl != q.tail[k] || lv != q.lvl[k]) {        // (never without a node: it has no successors)
            const int v = v0 + k * step;
            changed = true;
            q.tail[k] = tl; q.lvl[k] = lv;
            __hip_atomic_store(&a.tail[v], tl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.level[v], lv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.rem[v], q.c[k] + tl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (bad) hx_raise(a.status, HX_ERR_INDEX);
    return changed;
}

// sweep s (1, 2, ..) over the thread's nodes of the whole graph; over: the first begins with nothing but the costs
__device__ __forceinline__ bool hx_cp_sweep(const CpArgs &a, CgNodes &q, int first, int step, int s, bool over)
{
    const bool kept = a.n_nodes <= (long long)step * CG_NPT;      // all of them are in q from the first sweep on
    bool changed = false;
    for (long long v0 = first; v0 < a.n_nodes; v0 += (long long)step * CG_NPT) {
        if (!kept || s == 1) hx_cp_nodes_load(a, q, (int)v0, step, s == 1 && over);
        changed = hx_cp_nodes_sweep(a, q, (int)v0, step) || changed;
    }
    return changed;
}

__device__ __forceinline__ void hx_cp_sweep_init(const CpArgs &a, int first, int step)
{
    for (int v = first; v < a.n_nodes; v += step) {
        __hip_atomic_store(&a.tail[v], 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.rem[v], a.cost[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.level[v], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// A workflow's horizon by 16 lanes, or by a wavefront where workflows are large: thread `first` of `step`, both multiples
// of whole wavefronts but for the lane.
__device__ __forceinline__ void hx_cp_sweep_horizons(const CpArgs &a, int first, int step)
{
    const bool large = a.n_nodes > 64LL * a.n_wf;
    const int G = large ? HX_WAVE : 16, sub = first & (G - 1);
    // (whole wavefronts go round together: the reductions take every lane)
    for (int w0 = (first & ~(HX_WAVE - 1)) / G; w0 < a.n_wf; w0 += step / G) {
        const int w = w0 + (first & (HX_WAVE - 1)) / G;
        const int s = w < a.n_wf ? a.wf_ptr[w] : 0, e = w < a.n_wf ? a.wf_ptr[w + 1] : 0;
        float h = 0.0f;
        if (s < 0 || e > a.n_nodes || s > e) hx_raise(a.status, HX_ERR_INDEX);
        else {
#pragma unroll 4
            for (int v = s + sub; v < e; v += G) h = fmaxf(h, __hip_atomic_load(&a.rem[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
        h = large ? hx_wave_max(h) : -hx_lanes_min(-h, 16);
        if (sub == 0 && w < a.n_wf) __hip_atomic_store(&a.horizon[w], h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// All workgroups meet; *any: one of them came with `mark`.  target: arrivals so far, theirs included; seen: what the
// last meeting left (0 before the first).  The wait is bounded by `polls`: workgroups that are not on the chip yet (it may be full
// of other work) are waited for a while, then everybody gives up (false).
//
// Arrivals and marks are counted in the halves of one word; whoever completes the count passes it on to those who wait.
// No cache is written back or invalidated here (by every wavefront 60 us a meeting of 256 workgroups, by one wavefront
// of each 7): what passes from one workgroup to another inside the kernel -- rem, level and these words -- is stored and
// loaded by device-scope atomics alone, which the caches of an XCD do not hold back, and a store has arrived when
// its wavefront has waited for it.
__device__ __forceinline__ bool hx_grid_wait(int32_t *sync, int polls, unsigned target, bool mark, bool *any, unsigned long long *seen)
{
    __shared__ unsigned long long s_go;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // every wavefront's own stores have arrived
    mark = __syncthreads_or(mark);
    if (gridDim.x == 1) { *any = mark; return true; }
    if (threadIdx.x == 0) {
        unsigned long long *const count = (unsigned long long *)(sync + SY_COUNT), *const go = (unsigned long long *)(sync + SY_GO);
        const unsigned long long mine = 1ull + ((unsigned long long)mark << 32);
        unsigned long long now = __hip_atomic_fetch_add(count, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
        if ((unsigned)now == target) __hip_atomic_store(go, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            for (int i = 0; (unsigned)(now = __hip_atomic_load(go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != target; ++i) {
                if (i >= polls || ((i & 15) == 15 && __hip_atomic_load(&sync[SY_STUCK], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                    __hip_atomic_store(&sync[SY_STUCK], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    now = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
        s_go = now;
    }
    __syncthreads();
    const unsigned long long now = s_go;
    *any = (now >> 32) != (*seen >> 32);
    *seen = now;
    return now != 0;
}

// The whole graph, where the slices could not finish it: at most one workgroup per compute unit, a meeting of all of them a
// sweep (2 us with 40 workgroups, 3 with 256; a launch per sweep costs more than that also for graphs that need none).
// Should the workgroups not come together, the last one to leave does everything alone.
__global__ __launch_bounds__(CG_THREADS) void hx_cp_sweep_all_kernel(CpArgs a, int max_sweeps, int polls, int32_t *sync)
{
    __shared__ int s_last;
    if (sync[SY_AGAIN] == 0) return;
    const int first = blockIdx.x * CG_THREADS + threadIdx.x, step = gridDim.x * CG_THREADS;
    const bool over = sync[SY_OVER] != 0;
    CgNodes q;
    bool here = true, more = true;
    unsigned arrived = 0;
    unsigned long long seen = 0;
    if (over) {
        hx_cp_sweep_init(a, first, step);
        here = hx_grid_wait(sync, polls, arrived += gridDim.x, false, &more, &seen);
        more = true;
    }
    for (int s = 1; here && more && s <= max_sweeps; ++s)
        here = hx_grid_wait(sync, polls, arrived += gridDim.x, hx_cp_sweep(a, q, first, step, s, over), &more, &seen);
    if (here) {
        hx_cp_sweep_horizons(a, first, step);
        if (more && first == 0) hx_raise(a.status, HX_ERR_NOT_DAG);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) s_last = __hip_atomic_fetch_add(&sync[SY_LEFT], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    if (__hip_atomic_load(&sync[SY_STUCK], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
        hx_cp_sweep_init(a, threadIdx.x, CG_THREADS);
        more = true;
        for (int s = 1; more && s <= max_sweeps; ++s) {
            __threadfence();
            __syncthreads();
            more = __syncthreads_or(hx_cp_sweep(a, q, threadIdx.x, CG_THREADS, s, true));
        }
        __threadfence();
        __syncthreads();
        hx_cp_sweep_horizons(a, threadIdx.x, CG_THREADS);
        if (more && threadIdx.x == 0) hx_raise(a.status, HX_ERR_NOT_DAG);
    }
    __syncthreads();
    if (threadIdx.x < HX_SYNC_WORDS) __hip_atomic_store(&sync[threadIdx.x], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- incremental append ------------------------------------------------------------------

// workflow of a new node (-1: out of range)
__device__ __forceinline__ int hx_append_wf(const AppendArgs &a, int i)
{
    const int w = a.new_wf[i];
    return w >= 0 && w < a.cap_wf ? w : -1;
}

// first parent of the new node v (-1: none, or not a valid one)
__device__ __forceinline__ int hx_append_first_parent(const AppendArgs &a, int v)
{
    const int r0 = a.new_row_ptr[v - a.n_old], r1 = a.new_row_ptr[v - a.n_old + 1];
    if (r0 < 0 || r1 > a.n_new_edges || r0 >= r1) return -1;
    const int u = a.new_col[r0];
    return u >= 0 && u < v ? u : -1;
}

// First phase of an append: the new nodes' own entries.  The two list counters the append needs at zero (the
// one the walks append to, the one the first sweep after them clears) are cleared here: the walks are a launch
// of their own after this one, so no launch is spent on the counters.
// The horizons are raised by the walks, at the top of each workflow.
// COST: the nodes' standalone costs are not read but worked out here from their lengths, exactly as
// hx_node_cost_kernel does, and written to the caller's array as well (one launch less in front of the walks, where
// every launch of a round still waits for the host).
template <bool COST>
__global__ __launch_bounds__(256) void hx_append_init_kernel(AppendArgs a, NodeCostArgs nc)
{
    __shared__ CostTables s_tab;
    if constexpr (COST) {
        hx_cost_tables_fill(s_tab, nc, threadIdx.x);
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) { a.counters[a.czero] = 0; a.counters[a.cout] = 0; }
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < a.n_new; i += gridDim.x * blockDim.x) {
        const int v = a.n_old + i;
        unsigned bits;                                    // (no float may be the NaN)
        if constexpr (COST) {
            const float x = hx_node_cost_one(nc.m, s_tab, nc.T, nc.L_in[i], nc.L_out[i]);
            nc.cost[i] = x;
            bits = __float_as_uint(x);
        } else {
            bits = ((const unsigned *)a.new_cost)[i];
        }
        if (!hx_cost_ok(bits)) { hx_raise(a.status, HX_ERR_INVALID_ARG); bits = 0; }
        const float c = __uint_as_float(bits);
        int r0 = a.new_row_ptr[i], r1 = a.new_row_ptr[i + 1];
        const int w = hx_append_wf(a, i);
        if (w < 0) hx_raise(a.status, HX_ERR_INDEX);
        if (r0 < 0 || r1 > a.n_new_edges || r0 > r1) { hx_raise(a.status, HX_ERR_INDEX); r0 = r1 = min(max(r0, 0), a.n_new_edges); }
        a.rem[v] = c + 0.0f;                              // (-0.0, whose bits are above every number's, is 0)
        a.tail[v] = 0.0f; a.level[v] = 0; a.mark[v] = 0;
        a.prow[v + 1] = a.e_old + r1;
        int up[HX_CHAIN], second = -1;
        up[0] = -1;
        for (int e = r0; e < r1; ++e) {
            int u = a.new_col[e];
            if (u < 0 || u >= v) { hx_raise(a.status, HX_ERR_NOT_DAG); u = -1; }
            a.pcol[a.e_old + e] = u;
            if (e == r0) up[0] = u;
            if (e == r0 + 1) second = u;
        }
        // the first parents above: those of the nearest one that is not new lie beside it
        const int wf0 = up[0] < 0 ? -1 : up[0] < a.n_old ? a.rec[up[0]].y : hx_append_wf(a, up[0] - a.n_old);
        bool old = false;
#pragma unroll
        for (int k = 1; k < HX_CHAIN; ++k) {
            if (old) continue;
            const int p = up[k - 1];
            if (p >= a.n_old) { up[k] = hx_append_first_parent(a, p); continue; }
            int4 x = make_int4(-1, -1, -1, -1);
            if (p >= 0) x = a.chain[p];
            const int above[HX_CHAIN] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int j = k; j < HX_CHAIN; ++j) up[j] = above[j - k];
            old = true;
        }
        a.chain[v] = make_int4(up[0], up[1], up[2], up[3]);
        a.rec[v] = make_int4(__float_as_int(c), w, second, (up[0] < 0 || wf0 != w ? HX_NODE_TOP : 0) | (r1 - r0 > 2 ? HX_NODE_MANY : 0));
    }
}

template <bool REFRESH>
__global__ __launch_bounds__(256) void hx_append_relax_kernel(AppendArgs a)
{
    hx_append_relax_body<REFRESH>(a, (int)blockIdx.x, (int)gridDim.x);
}

__global__ void hx_append_finish_kernel(AppendArgs a)
{
    if (threadIdx.x == 0 && a.counters[a.cin] != 0) hx_raise(a.status, HX_ERR_CAPACITY);
}

// The remaining sweeps in one workgroup: after a few grid-wide sweeps the lists
// are short, and what is left is a chain of dependent steps -- one launch loops
// over them until the list is empty (or `sweeps` steps are done) instead of one
// launch per step.  Every value another thread may have written is read with a
// device-scope load.
__global__ __launch_bounds__(1024) void hx_append_tail_kernel(AppendArgs a, int32_t *list0, int32_t *list1,
                                                              int first, int sweeps)
{
    __shared__ int s_n;
    for (int s = first; s < first + sweeps; ++s) {
        a.cin = (s + 1) % 3; a.cout = (s + 2) % 3; a.czero = s % 3;
        a.list_in = (s & 1) ? list1 : list0;
        a.list_out = (s & 1) ? list0 : list1;
        a.epoch += 1;
        if (threadIdx.x == 0) {
            s_n = __hip_atomic_load(&a.counters[a.cin], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.counters[a.czero], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        const int n = s_n;
        if (n == 0) break;                                   // uniform: nothing left to propagate
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const int u = __hip_atomic_load(&a.list_in[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float tl = __hip_atomic_load(&a.tail[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int lv = __hip_atomic_load(&a.level[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int4 me = a.rec[u];
            const float r = hx_node_rec_cost(me) + tl;
            a.rem[u] = r;
            if (me.y >= 0) hx_raise_max_f32(&a.horizon[me.y], r);
            for (int e = a.prow[u]; e < a.prow[u + 1]; ++e) {
                int q = a.pcol[e];
                if (q >= 0) hx_push_parent(a, q, r, lv);
            }
        }
        __threadfence();
        __syncthreads();
    }
    // the list the last step wrote must be empty, or the depth limit was too small
    if (threadIdx.x == 0) {
        const int last = (first + sweeps + 1) % 3;
        if (__hip_atomic_load(&a.counters[last], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 &&
            s_n != 0) hx_raise(a.status, HX_ERR_CAPACITY);
    }
}

// Cost of existing nodes replaced by observed values (an id outside the graph, or a cost below 0, is skipped and reported), and what the costs
// determine back to its starting point: no horizons, no tails, those of nodes with children marked as not reached.
__global__ __launch_bounds__(256) void hx_refresh_begin_kernel(AppendArgs a, int n, const int32_t *ids, const float *value, int n_wf)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const int v = ids[i];
        if (v < 0 || v >= a.n_new) hx_raise(a.status, HX_ERR_INDEX);
        else if (const int bits = ((const int *)value)[i]; hx_cost_ok((unsigned)bits)) a.rec[v].x = bits;
        else hx_raise(a.status, HX_ERR_INVALID_ARG);
    }
    if (i < a.n_new) ((int *)a.tail)[i] = a.level[i] > 0 ? -1 : 0;
    if (i < n_wf) a.horizon[i] = 0.0f;
    if (i < 3) a.counters[i] = 0;
}

// rem from the tails, and the horizons from the tops of the workflows
__global__ __launch_bounds__(256) void hx_refresh_end_kernel(AppendArgs a)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= a.n_new) return;
    const int4 me = a.rec[v];
    const int t = ((const int *)a.tail)[v];
    if (t < 0) a.tail[v] = 0.0f;                          // (never reached: the sweeps ran out, which the status says)
    const float r = hx_node_rec_cost(me) + __int_as_float(max(t, 0));
    a.rem[v] = r;
    if ((me.w & HX_NODE_TOP) && me.y >= 0) hx_raise_max_f32(&a.horizon[me.y], r);
}

// An empty graph: the horizon of every workflow 0, the first row's bound 0, the list counters 0.  (One launch: behind the wait for
// the device the host is what the next kernels wait for.)
__global__ __launch_bounds__(256) void hx_reserve_kernel(float *horizon, size_t n_wf, int32_t *row_ptr, int32_t *counters)
{
    const size_t at = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (at == 0) row_ptr[0] = 0;
    if (at < 4) counters[at] = 0;
    for (size_t i = at; i < n_wf; i += (size_t)gridDim.x * blockDim.x) horizon[i] = 0.0f;
}

template <typename T>
int dev_alloc(hx_ctx *ctx, T **p, size_t n)
{
    *p = nullptr;
    HX_HIP(ctx, hipMalloc((void **)p, (n ? n : 1) * sizeof(T)));
    return HX_OK;
}

void dag_free(HxDagStore &g)
{
    void *ptrs[] = {g.rec, g.chain, g.rem, g.tail, g.horizon, g.level, g.parent_row_ptr, g.parent_col,
                    g.mark, g.list[0], g.list[1], g.counters};
    for (void *p : ptrs) if (p) (void)hipFree(p);
    g = HxDagStore{};
}

}  // namespace

void hx_dag_release(hx_ctx *ctx) { dag_free(ctx->dag); }

namespace {

// the argument checks of the standalone cost, and its kernel arguments
int node_cost_args(hx_ctx *ctx, const hx_model *model, int32_t n, const int32_t *L_in, const int32_t *L_out,
                   int32_t n_types, const float *type_flops, const float *type_hbm_bw, const hx_links *links, float *cost,
                   NodeCostArgs *out)
{
    HX_REQUIRE(ctx, model && links && links->bw && type_flops && type_hbm_bw, HX_ERR_INVALID_ARG, "NULL table");
    HX_REQUIRE(ctx, n >= 0, HX_ERR_INVALID_ARG, "negative n");
    HX_REQUIRE(ctx, n_types >= 1 && n_types <= HX_MAX_TYPES && links->n_types == n_types, HX_ERR_SHAPE,
               "n_types %d (links %d) outside 1..%d", n_types, links->n_types, HX_MAX_TYPES);
    HX_REQUIRE(ctx, n == 0 || (L_in && L_out && cost), HX_ERR_INVALID_ARG, "NULL array");
    NodeCostArgs a{};
    a.m = HxModelF{model->kv_bytes_per_token, model->flops_per_token, model->attn_flops_per_token2,
                   model->weight_bytes, model->nominal_batch};
    a.n = n; a.T = n_types; a.L_in = L_in; a.L_out = L_out; a.tF = type_flops; a.tB = type_hbm_bw;
    a.bw = links->bw; a.lat = links->latency; a.cost = cost;
    *out = a;
    return HX_OK;
}

}  // namespace

extern "C" int hx_node_cost(hx_ctx *ctx, const hx_model *model, int32_t n,
                            const int32_t *L_in, const int32_t *L_out,
                            int32_t n_types, const float *type_flops, const float *type_hbm_bw,
                            const hx_links *links, float *cost, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    NodeCostArgs a{};
    if (int rc = node_cost_args(ctx, model, n, L_in, L_out, n_types, type_flops, type_hbm_bw, links, cost, &a)) return rc;
    if (n == 0) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    // Four nodes a thread where there are many (launches in a graph, one and four a thread: 262144 nodes of 4 classes 3.1 and 3.5 us, 400000
    // 3.6 and 3.5; 400000 of 5 and of 8 4.1 and 4.8, 5.3 and 6.7; 786432 5.3 and 5.3, 7.8 and 7.3), at most eight workgroups a
    // compute unit.  More than four classes of few nodes: all pairs at once (65536 nodes of 5, 6, 7, 8 classes 3.0, 3.0, 3.0, 3.1 us, one
    // class after the other 3.1, 3.3, 3.7, 4.0; 131072 3.3, 3.4, 3.4, 3.5 and 3.2, 3.4, 3.8, 4.1; 200000 5.1 to 5.6 and 3.4 to 4.4).
    const int nn = n >= ctx->num_cu * (n_types > 4 ? 3072 : 1536) ? 4 : 1;
    const bool at_once = n_types > 4 && n <= ctx->num_cu * (n_types > 5 ? 512 : 256);
    int grid = (int)(((long long)n + 256 * nn - 1) / (256 * nn));
    grid = grid > ctx->num_cu * 8 ? ctx->num_cu * 8 : grid;
    hipStream_t stream = (hipStream_t)stream_;
    if (at_once) hx_node_cost_kernel<1, kT, true><<<grid, 256, 0, stream>>>(a);
    else if (nn == 1) hx_node_cost_kernel<1, kT><<<grid, 256, 0, stream>>>(a);
    else if (n_types <= 4) hx_node_cost_kernel<4, 4><<<grid, 256, 0, stream>>>(a);
    else hx_node_cost_kernel<4, kT><<<grid, 256, 0, stream>>>(a);
    return hx_check_launch(ctx, "hx_node_cost_kernel");
}

// Workflows a wavefront takes (hx_cp_wave), one each as long as that fills the chip with wavefronts and no more than fit its lanes.
// 0: workgroups take slices, where workflows are too large on the average, or nodes are more than `most` a compute unit.
static int wave_workflows(const hx_ctx *ctx, int n_nodes, int n_wf, int most)
{
    if (n_wf == 0 || n_nodes > 48LL * n_wf || n_nodes > (long long)most * ctx->num_cu) return 0;
    const long long fit = n_nodes > 0 ? 56LL * n_wf / n_nodes : 32, spread = n_wf / (8 * ctx->num_cu);
    const long long n = fit < spread ? fit : spread;
    return (int)(n < 1 ? 1 : (n > 32 ? 32 : n));
}
// Launches in a graph, slices and wavefronts (us).  With the node cost of 4 classes: 20000 nodes 10.1 and 6.2, 82000 10.7 and 6.8, 200000
// 11.2 and 11.6, 1.8 million 29 and 67; of 8 classes 200000 15.8 and 14.0, 240000 in workflows of 8 13.8 and 15.6.  Sweeps: 20000 12.8 and
// 7.3, 200000 14.0 and 10.0, 320000 15.6 and 13.4, 440000 15.9 and 15.7, 600000 18.0 and 19.8.  1000 workflows of 30 to 60 nodes 14.5 and 6.4;
// of 24 to 70, a tenth of which are too large, 13.2 and 12.5, sweeps 39.7 and 33.7; 1000 of 10 to 30 with one of 100 in each 20th 15.0 and 14.5, sweeps 36 and 37.
constexpr int CW_MOST_COST = 384, CW_MOST_SWEEPS = 1536;

extern "C" int hx_critical_path(hx_ctx *ctx, int32_t n_nodes, int32_t n_edges,
                                const int32_t *succ_row_ptr, const int32_t *succ_col_idx,
                                const float *node_cost, int32_t n_wf, const int32_t *wf_ptr,
                                int32_t max_sweeps,
                                float *rem, float *tail, int32_t *level, float *horizon, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HX_REQUIRE(ctx, n_nodes >= 0 && n_edges >= 0 && n_wf >= 0 && max_sweeps >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, max_sweeps < HX_SWEEP_LIMIT, HX_ERR_SHAPE, "max_sweeps beyond %d", HX_SWEEP_LIMIT - 1);
    HX_REQUIRE(ctx, succ_row_ptr && wf_ptr, HX_ERR_INVALID_ARG, "NULL row_ptr or wf_ptr");
    HX_REQUIRE(ctx, n_edges == 0 || succ_col_idx, HX_ERR_INVALID_ARG, "NULL col_idx");
    HX_REQUIRE(ctx, n_nodes == 0 || (node_cost && rem && tail && level), HX_ERR_INVALID_ARG, "NULL node array");
    HX_REQUIRE(ctx, n_wf == 0 || horizon, HX_ERR_INVALID_ARG, "NULL horizon");
    if (n_wf == 0 && (n_nodes == 0 || max_sweeps == 0)) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;
    CpArgs a{n_nodes, n_edges, n_wf, succ_row_ptr, succ_col_idx, wf_ptr, node_cost, rem, tail, horizon, level,
             ctx->d_status};
    if (max_sweeps == 0) {
        // workflows per block: as many as fit the staged slice at the average workflow size
        long long fit = n_nodes > 0 ? (long long)(CP_NMAX * 41 / 50) * n_wf / n_nodes : CP_WPB;
        const int wpb = (int)(fit < 1 ? 1 : (fit > CP_WPB ? CP_WPB : fit));
        const int grid = (n_wf + wpb - 1) / wpb;
        // results of 12 MB and more are streamed out past the caches
        if (n_nodes >= (1 << 20)) hx_cp_local_kernel<true><<<grid, CP_THREADS, 0, stream>>>(a, wpb);
        else hx_cp_local_kernel<false><<<grid, CP_THREADS, 0, stream>>>(a, wpb);
        return hx_check_launch(ctx, "hx_cp_local_kernel");
    }
    // Slices: workflows enough for two thirds of a workgroup's room, but no more than it takes to give every compute unit
    // a slice; without workflows or nodes there is nothing to slice, and the second kernel is told to run.
    long long fit = n_nodes > 0 && n_wf > 0 ? (long long)(CS_NMAX * 2 / 3) * n_wf / n_nodes : 1;
    const long long spread = (n_wf + ctx->num_cu - 1) / ctx->num_cu;
    fit = fit > spread ? spread : fit;
    const int wpv = wave_workflows(ctx, n_nodes, n_wf, CW_MOST_SWEEPS);
    const int wpb = wpv ? wpv * (CS_THREADS / HX_WAVE) : (int)(fit < 1 ? 1 : fit);
    const int n_slices = n_wf > 0 ? (n_wf + wpb - 1) / wpb : 1;
    if (wpv) hx_cp_sweep_slices_kernel<true><<<n_slices, CS_THREADS, 0, stream>>>(a, wpb, wpv, max_sweeps, ctx->d_sync);
    else hx_cp_sweep_slices_kernel<false><<<n_slices, CS_THREADS, 0, stream>>>(a, wpb, 0, max_sweeps, ctx->d_sync);
    if (int rc = hx_check_launch(ctx, "hx_cp_sweep_slices_kernel")) return rc;
    const long long most = n_nodes > n_wf ? n_nodes : n_wf;      // (workflows may be empty)
    int grid = (int)((most + CG_THREADS - 1) / CG_THREADS);
    grid = grid > ctx->num_cu ? ctx->num_cu : (grid < 1 ? 1 : grid);
    hx_cp_sweep_all_kernel<<<grid, CG_THREADS, 0, stream>>>(a, max_sweeps, ctx->sweep_polls, ctx->d_sync);
    return hx_check_launch(ctx, "hx_cp_sweep_all_kernel");
}

// for tests: how long a workgroup of the sweeps waits for the others (0: all but the last to arrive give up at once)
extern "C" int hx_test_sweep_polls(hx_ctx *ctx, int polls)
{
    if (!ctx || polls < 0) return HX_ERR_INVALID_ARG;
    ctx->sweep_polls = polls;
    return HX_OK;
}

int hx_horizons_plan(hx_ctx *ctx, const hx_model *model, int32_t n_nodes, int32_t n_edges,
                     const int32_t *succ_row_ptr, const int32_t *succ_col_idx,
                     const int32_t *L_in, const int32_t *L_out,
                     int32_t n_types, const float *type_flops, const float *type_hbm_bw, const hx_links *links,
                     int32_t n_wf, const int32_t *wf_ptr,
                     float *node_cost, float *rem, float *tail, int32_t *level, float *horizon, HxHorizonsPlan *plan)
{
    HX_REQUIRE(ctx, model && links && links->bw && type_flops && type_hbm_bw, HX_ERR_INVALID_ARG, "NULL table");
    HX_REQUIRE(ctx, n_nodes >= 0 && n_edges >= 0 && n_wf >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, n_types >= 1 && n_types <= HX_MAX_TYPES && links->n_types == n_types, HX_ERR_SHAPE,
               "n_types %d (links %d) outside 1..%d", n_types, links->n_types, HX_MAX_TYPES);
    HX_REQUIRE(ctx, succ_row_ptr && wf_ptr, HX_ERR_INVALID_ARG, "NULL row_ptr or wf_ptr");
    HX_REQUIRE(ctx, n_edges == 0 || succ_col_idx, HX_ERR_INVALID_ARG, "NULL col_idx");
    HX_REQUIRE(ctx, n_nodes == 0 || (L_in && L_out && node_cost && rem && tail && level), HX_ERR_INVALID_ARG, "NULL node array");
    HX_REQUIRE(ctx, n_wf == 0 || horizon, HX_ERR_INVALID_ARG, "NULL horizon");
    *plan = HxHorizonsPlan{};
    if (n_wf == 0) return HX_OK;
    plan->a = CpArgs{n_nodes, n_edges, n_wf, succ_row_ptr, succ_col_idx, wf_ptr, node_cost, rem, tail, horizon, level,
                     ctx->d_status};
    NodeCostArgs nc{};
    nc.m = HxModelF{model->kv_bytes_per_token, model->flops_per_token, model->attn_flops_per_token2,
                    model->weight_bytes, model->nominal_batch};
    nc.n = n_nodes; nc.T = n_types; nc.L_in = L_in; nc.L_out = L_out; nc.tF = type_flops; nc.tB = type_hbm_bw;
    nc.bw = links->bw; nc.lat = links->latency; nc.cost = node_cost;
    plan->nc = nc;
    // workflows per block: as many as fit the staged slice at the average workflow size, but no more
    // than it takes to give every compute unit a block (a thread evaluates the cost of each of its nodes)
    long long fit = n_nodes > 0 ? (long long)(CP_NMAX_COST * 41 / 50) * n_wf / n_nodes : CP_WPB;
    const long long spread = n_wf / ctx->num_cu;
    fit = fit > spread ? (spread < 1 ? 1 : spread) : fit;
    plan->wpb = (int)(fit < 1 ? 1 : (fit > CP_WPB ? CP_WPB : fit));
    plan->grid = (n_wf + plan->wpb - 1) / plan->wpb;
    plan->wpv = wave_workflows(ctx, n_nodes, n_wf, CW_MOST_COST);
    return HX_OK;
}

extern "C" int hx_horizons(hx_ctx *ctx, const hx_model *model, int32_t n_nodes, int32_t n_edges,
                           const int32_t *succ_row_ptr, const int32_t *succ_col_idx,
                           const int32_t *L_in, const int32_t *L_out,
                           int32_t n_types, const float *type_flops, const float *type_hbm_bw, const hx_links *links,
                           int32_t n_wf, const int32_t *wf_ptr,
                           float *node_cost, float *rem, float *tail, int32_t *level, float *horizon, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HxHorizonsPlan plan;
    if (int rc = hx_horizons_plan(ctx, model, n_nodes, n_edges, succ_row_ptr, succ_col_idx, L_in, L_out, n_types, type_flops,
                                  type_hbm_bw, links, n_wf, wf_ptr, node_cost, rem, tail, level, horizon, &plan))
        return rc;
    if (plan.grid == 0) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    // As many workflows a workgroup as the slices it may fall back to take in one run (40000 workflows of 2 nodes, some of 65 among them
    // 15.6 us, 18.4 in runs of 64 and 12; without them 6.2 either way).  Slices where there are no edges to speak of: they take
    // a lane a workflow then, without LDS (16384 single nodes 4.3 us, by wavefronts 5.4).
    const int waves = CP_THREADS / HX_WAVE, most = CP_WPB / waves;
    const int wpv = n_edges < CP_DEG ? 0 : (plan.wpv < most ? plan.wpv : most);
    const int wpb = wpv ? wpv * waves : plan.wpb;
    const int grid = (n_wf + wpb - 1) / wpb;
    if (wpv) hx_cp_cost_kernel<true><<<grid, CP_THREADS, 0, (hipStream_t)stream_>>>(plan.a, plan.nc, wpb, wpv);
    else hx_cp_cost_kernel<false><<<grid, CP_THREADS, 0, (hipStream_t)stream_>>>(plan.a, plan.nc, wpb, 0);
    return hx_check_launch(ctx, "hx_cp_cost_kernel");
}

extern "C" int hx_dag_reserve(hx_ctx *ctx, int32_t max_nodes, int32_t max_edges, int32_t max_wf,
                              int32_t max_depth, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HX_REQUIRE(ctx, max_nodes >= 0 && max_edges >= 0 && max_wf >= 0 && max_depth >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, max_depth <= 4096, HX_ERR_SHAPE, "max_depth beyond 4096");
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;
    HxDagStore &g = ctx->dag;
    int rc = HX_OK;
    const size_t N = (size_t)max_nodes, E = (size_t)max_edges, W = (size_t)max_wf;
    // A store that is large enough and not more than twice as large as asked for is kept: freeing and allocating its 12
    // arrays costs some 350 us, a third of a session of eight rounds (1120 -> 786 us).
    auto keeps = [](int32_t have, size_t want) { return (size_t)have >= want && (size_t)have <= 2 * want; };
    const bool keep = g.rec && keeps(g.room_nodes, N) && keeps(g.room_edges, E) && keeps(g.room_wf, W);
    // Whatever is still at work on the old graph, on any stream, is waited for: by the device where its arrays stay, as
    // freeing them does otherwise; nothing but this stream where there are none.
    if (keep) HX_HIP(ctx, hipDeviceSynchronize());
    else {
        HX_HIP(ctx, hipStreamSynchronize(stream));
        dag_free(g);
    }
    if (!keep && ((rc = dev_alloc(ctx, &g.rec, N)) || (rc = dev_alloc(ctx, &g.chain, N)) || (rc = dev_alloc(ctx, &g.rem, N)) || (rc = dev_alloc(ctx, &g.tail, N)) ||
        (rc = dev_alloc(ctx, &g.horizon, W)) || (rc = dev_alloc(ctx, &g.level, N)) ||
        (rc = dev_alloc(ctx, &g.parent_row_ptr, N + 1)) || (rc = dev_alloc(ctx, &g.parent_col, E)) ||
        (rc = dev_alloc(ctx, &g.mark, N)) || (rc = dev_alloc(ctx, &g.list[0], N)) ||
        (rc = dev_alloc(ctx, &g.list[1], N)) || (rc = dev_alloc(ctx, &g.counters, (size_t)4)))) {
        dag_free(g);
        return rc;
    }
    if (!keep) { g.room_nodes = max_nodes; g.room_edges = max_edges; g.room_wf = max_wf; }
    g.cap_nodes = max_nodes; g.cap_edges = max_edges; g.cap_wf = max_wf; g.max_depth = max_depth;
    g.n_nodes = 0; g.n_edges = 0; g.epoch = 0;
    hx_reserve_kernel<<<256, 256, 0, stream>>>(g.horizon, W, g.parent_row_ptr, g.counters);      // (a kernel, no memset nodes)
    return hx_check_launch(ctx, "hx_reserve_kernel");
}

namespace {

// The append's first kernel.  nc: NULL, or the arguments of the standalone cost of the new nodes, which that kernel
// then works out itself (new_cost is nc->cost then, written as well as used).  plan->grid == 0: nothing to append.
int dag_append_begin(hx_ctx *ctx, int32_t n_new, int32_t n_new_edges, const int32_t *parent_row_ptr, const int32_t *parent_col_idx,
                     const float *new_cost, const int32_t *new_wf, const NodeCostArgs *nc, HxAppendPlan *plan, hipStream_t stream)
{
    *plan = HxAppendPlan{};
    HxDagStore &g = ctx->dag;
    HX_REQUIRE(ctx, g.rec, HX_ERR_INVALID_ARG, "hx_dag_reserve has not been called");
    HX_REQUIRE(ctx, n_new >= 0 && n_new_edges >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, n_new == 0 || (parent_row_ptr && new_cost && new_wf), HX_ERR_INVALID_ARG, "NULL array");
    HX_REQUIRE(ctx, n_new_edges == 0 || parent_col_idx, HX_ERR_INVALID_ARG, "NULL parent_col_idx");
    HX_REQUIRE(ctx, (long long)g.n_nodes + n_new <= g.cap_nodes, HX_ERR_CAPACITY,
               "%d + %d nodes beyond the reserved %d", g.n_nodes, n_new, g.cap_nodes);
    HX_REQUIRE(ctx, (long long)g.n_edges + n_new_edges <= g.cap_edges, HX_ERR_CAPACITY,
               "%d + %d edges beyond the reserved %d", g.n_edges, n_new_edges, g.cap_edges);
    if (n_new == 0) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);

    AppendArgs a{};
    a.n_old = g.n_nodes; a.n_new = n_new; a.e_old = g.n_edges; a.n_new_edges = n_new_edges; a.cap_wf = g.cap_wf;
    a.new_row_ptr = parent_row_ptr; a.new_col = parent_col_idx; a.new_wf = new_wf; a.new_cost = new_cost;
    a.rec = g.rec; a.chain = g.chain; a.rem = g.rem; a.tail = g.tail; a.horizon = g.horizon;
    a.level = g.level; a.prow = g.parent_row_ptr; a.pcol = g.parent_col; a.mark = g.mark;
    a.counters = g.counters; a.status = ctx->d_status;

    int grid = (n_new + 255) / 256;
    grid = grid > ctx->num_cu * 8 ? ctx->num_cu * 8 : grid;
    a.cin = 0; a.cout = 1; a.czero = 2; a.epoch = ++g.epoch;
    a.list_in = g.list[1]; a.list_out = g.list[0];
    if (nc) hx_append_init_kernel<true><<<grid, 256, 0, stream>>>(a, *nc);
    else hx_append_init_kernel<false><<<grid, 256, 0, stream>>>(a, NodeCostArgs{});
    if (int rc = hx_check_launch(ctx, "hx_append_init_kernel")) return rc;
    plan->a = a; plan->grid = grid; plan->n_new = n_new; plan->n_new_edges = n_new_edges;
    return HX_OK;
}

int dag_append(hx_ctx *ctx, int32_t n_new, int32_t n_new_edges, const int32_t *parent_row_ptr, const int32_t *parent_col_idx,
               const float *new_cost, const int32_t *new_wf, const NodeCostArgs *nc, hipStream_t stream)
{
    HxAppendPlan plan;
    if (int rc = dag_append_begin(ctx, n_new, n_new_edges, parent_row_ptr, parent_col_idx, new_cost, new_wf, nc, &plan, stream)) return rc;
    if (plan.grid == 0) return HX_OK;
    if (int rc = hx_dag_append_walks(ctx, &plan, stream)) return rc;
    return hx_dag_append_end(ctx, &plan, stream);
}

}  // namespace

// the walks of an append that has begun, as a launch of their own
int hx_dag_append_walks(hx_ctx *ctx, const HxAppendPlan *plan, void *stream)
{
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hx_append_relax_kernel<false><<<plan->grid, 256, 0, (hipStream_t)stream>>>(plan->a);
    return hx_check_launch(ctx, "hx_append_relax_kernel");
}

// what follows the walks: what they handed over (normally nothing) is finished level by level in one workgroup --
// sweep k reads the list sweep k-1 wrote, max_depth sweeps reach every ancestor -- and the graph has grown
int hx_dag_append_end(hx_ctx *ctx, const HxAppendPlan *plan, void *stream_)
{
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;
    HxDagStore &g = ctx->dag;
    AppendArgs a = plan->a;
    if (g.max_depth > 0) {
        a.epoch = g.epoch;                       // the loop advances it once per step
        hx_append_tail_kernel<<<1, 1024, 0, stream>>>(a, g.list[0], g.list[1], 0, g.max_depth);
        g.epoch += (uint32_t)g.max_depth;
    } else {
        a.cin = 1;
        hx_append_finish_kernel<<<1, 64, 0, stream>>>(a);
    }
    if (int rc = hx_check_launch(ctx, "hx_dag_append kernels")) return rc;
    g.n_nodes += plan->n_new;
    g.n_edges += plan->n_new_edges;
    return HX_OK;
}

extern "C" int hx_dag_append(hx_ctx *ctx, int32_t n_new, int32_t n_new_edges,
                             const int32_t *parent_row_ptr, const int32_t *parent_col_idx,
                             const float *new_cost, const int32_t *new_wf, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    return dag_append(ctx, n_new, n_new_edges, parent_row_ptr, parent_col_idx, new_cost, new_wf, nullptr, (hipStream_t)stream_);
}

// hx_node_cost of the new nodes followed by the first kernel of hx_dag_append, the cost worked out by that kernel: the
// same checks and the same results as the two calls, one launch less (for hx_round, which goes on with
// hx_dag_append_walks -- or takes the walks into its search's launch -- and hx_dag_append_end)
int hx_dag_append_begin(hx_ctx *ctx, const hx_model *model, int32_t n_new, int32_t n_new_edges,
                        const int32_t *parent_row_ptr, const int32_t *parent_col_idx,
                        const int32_t *new_L_in, const int32_t *new_L_out,
                        int32_t n_types, const float *type_flops, const float *type_hbm_bw, const hx_links *links,
                        float *new_cost, const int32_t *new_wf, HxAppendPlan *plan, void *stream_)
{
    *plan = HxAppendPlan{};
    NodeCostArgs nc{};
    if (int rc = node_cost_args(ctx, model, n_new, new_L_in, new_L_out, n_types, type_flops, type_hbm_bw, links, new_cost, &nc))
        return rc;
    return dag_append_begin(ctx, n_new, n_new_edges, parent_row_ptr, parent_col_idx, new_cost, new_wf, &nc, plan, (hipStream_t)stream_);
}

// A refresh of a graph of more than this many nodes for every compute unit starts at the nodes without children, if it has at most
// two edges a node; else every node walks.  Fewer walks count where the device cannot work on all of them at a time: whole refreshes (us) with every
// node and so, 812 K nodes of a live system's workflows 69 and 64; workflows of 20, 800 K nodes in trees 65 and 37, of 1.35 edges a node 156 and 83, of
// 1.75 238 and 157, of 2.05 254 and 176; 200 K 27 and 22, 37 and 28 (1.25), 68 and 59 (1.65); 120 K 19 and 17, 29 and 24, 42 and 41; 20 K 16 and 15.  But a walk
// from below reaches a node once for every path that still raises it, one thread for all above a leaf, and neither count says how many
// paths there are: 6 graphs of 1000 nodes, 1.2 edges each, 0.55 and 4.6 ms, 20 of them 0.5 and 1.4, of 1.9 edges 3.7 and 8.0, 20 of 40 layers of 10
// 3.3 and 7.0; 100 graphs of 200 nodes, 1.4 edges, 150 and 218 us, 1000 of these 265 and 258.  Hence where it is the smaller graphs that would lose, the
// line lies where their gain is small: 2 to 5 us below it.
constexpr int REFRESH_LEAVES_NODES = 512;

extern "C" int hx_dag_set_cost(hx_ctx *ctx, int32_t n, const int32_t *node_ids, const float *cost, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HxDagStore &g = ctx->dag;
    HX_REQUIRE(ctx, g.rec, HX_ERR_INVALID_ARG, "hx_dag_reserve has not been called");
    HX_REQUIRE(ctx, n >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, n == 0 || (node_ids && cost), HX_ERR_INVALID_ARG, "NULL array");
    if (n == 0 || g.n_nodes == 0) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;
    // a cost may have gone down, so nothing can be kept (levels do not depend on costs and stay)
    AppendArgs a{};
    a.n_old = 0; a.n_new = g.n_nodes; a.cap_wf = g.cap_wf;
    a.rec = g.rec; a.chain = g.chain; a.rem = g.rem; a.tail = g.tail; a.horizon = g.horizon;
    a.level = g.level; a.prow = g.parent_row_ptr; a.pcol = g.parent_col; a.mark = g.mark;
    a.counters = g.counters; a.status = ctx->d_status;
    a.cin = 0; a.cout = 1; a.czero = 2; a.epoch = ++g.epoch;
    a.list_in = g.list[1]; a.list_out = g.list[0];
    a.leaves = g.n_nodes > ctx->num_cu * REFRESH_LEAVES_NODES && g.n_edges / 2 <= g.n_nodes;
    int m = g.n_nodes > g.cap_wf ? g.n_nodes : g.cap_wf;
    m = m > n ? m : n;
    hx_refresh_begin_kernel<<<(int)(((long long)m + 255) / 256), 256, 0, stream>>>(a, n, node_ids, cost, g.cap_wf);
    int grid = (g.n_nodes + 255) / 256;
    grid = grid > ctx->num_cu * 8 ? ctx->num_cu * 8 : grid;
    hx_append_relax_kernel<true><<<grid, 256, 0, stream>>>(a);
    if (g.max_depth > 0) {
        a.epoch = g.epoch;
        hx_append_tail_kernel<<<1, 1024, 0, stream>>>(a, g.list[0], g.list[1], 0, g.max_depth);
        g.epoch += (uint32_t)g.max_depth;
    } else {
        a.cin = 1;
        hx_append_finish_kernel<<<1, 64, 0, stream>>>(a);
    }
    hx_refresh_end_kernel<<<(int)(((long long)g.n_nodes + 255) / 256), 256, 0, stream>>>(a);
    return hx_check_launch(ctx, "hx_dag_set_cost kernels");
}

extern "C" int hx_dag_view(hx_ctx *ctx, const float **rem, const float **tail, const int32_t **level,
                           const float **horizon, int32_t *n_nodes)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HxDagStore &g = ctx->dag;
    HX_REQUIRE(ctx, g.rec, HX_ERR_INVALID_ARG, "hx_dag_reserve has not been called");
    if (rem) *rem = g.rem;
    if (tail) *tail = g.tail;
    if (level) *level = g.level;
    if (horizon) *horizon = g.horizon;
    if (n_nodes) *n_nodes = g.n_nodes;
    return HX_OK;
}
