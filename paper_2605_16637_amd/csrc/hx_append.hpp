// Device code of the incremental append's walks (Sec. 4.1, online reveal; Sec. 5.1, the horizon is refreshed at every
// reveal), shared by the append's own kernels in hx_dag.hip and by the scheduling round's merged launch in
// hx_score.hip.
#pragma once

#include "hx_common.hpp"

// A node of the graph store, 16 bytes: cost (bits), workflow (-1: none), second parent (-1: none), flags.
constexpr int HX_NODE_TOP = 1;    // no first parent, or one of another workflow: nothing above it stands for it in its workflow's horizon
constexpr int HX_NODE_MANY = 2;   // more than two parents: the others are read from its row of the parent lists

// The first parents above a node (its own, that one's, ...; -1 beyond the last), kept beside it: 16 bytes.
constexpr int HX_CHAIN = 4;

struct AppendArgs {
    int n_old, n_new, e_old, n_new_edges, cap_wf;
    const int32_t *new_row_ptr, *new_col, *new_wf;
    const float *new_cost;
    int4 *rec, *chain;
    float *rem, *tail, *horizon;
    int32_t *level, *prow, *pcol, *mark;
    int32_t *list_in, *list_out;
    int32_t *counters;      // [0..2] rotating list sizes
    int leaves;             // a refresh: only nodes without children walk
    int cin, cout, czero;   // which counter is read, appended to, cleared
    uint32_t epoch;
    int32_t *status;
};

__device__ __forceinline__ float hx_node_rec_cost(const int4 &rec) { return __int_as_float(rec.x); }

// A cost a node can have: not below 0, and a number.  By its bits, above +inf's of which lie the NaNs and everything with a sign
// (-0.0 is 0).  Tails and rems are raised on their bits, so no other cost may get into the graph.
__device__ __forceinline__ bool hx_cost_ok(unsigned bits) { return bits <= 0x7f800000u || bits == 0x80000000u; }

// non-negative fp32 values order like their bit patterns
__device__ __forceinline__ bool hx_raise_max_f32(float *addr, float v)
{
    unsigned old = atomicMax((unsigned *)addr, __float_as_uint(v));
    return __float_as_uint(v) > old;
}

// A tail as signed bits: costs have none below zero, and -1, less than any, marks a tail that a refresh has yet to reach.
__device__ __forceinline__ bool hx_raise_tail(const AppendArgs &a, int u, float v)
{
    return __float_as_int(v) > atomicMax((int *)&a.tail[u], __float_as_int(v));
}

// push the (new) rem and level of node v to its parent u; enqueue u if it grew.  The lanes of a
// wavefront that enqueue at the same moment take their list slots with one atomic between them
// (the list counter is a single address: one atomic per lane would serialise the whole sweep).
// The list entry is written with a device-scope store: later steps of the single-workgroup loop read the list back.
__device__ __forceinline__ void hx_push_parent(const AppendArgs &a, int u, float rem_v, int level_v)
{
    bool grew = hx_raise_tail(a, u, rem_v);
    int old = atomicMax(&a.level[u], level_v + 1);
    grew = grew || (level_v + 1 > old);
    const bool want = grew && (uint32_t)atomicExch(&a.mark[u], (int)a.epoch) != a.epoch;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(want);      // of the lanes active here
    if (m) {
        const int lane = (int)(threadIdx.x & (HX_WAVE - 1));
        const int leader = __ffsll((long long)m) - 1;
        int base = 0;
        if (lane == leader) base = atomicAdd(&a.counters[a.cout], __popcll(m));
        base = __shfl(base, leader);
        if (want) {
            const int slot = base + __popcll(m & ((1ull << lane) - 1ull));   // at most one entry per node and sweep: never beyond cap_nodes
            __hip_atomic_store(&a.list_out[slot], u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// node u onto the worklist of the next sweep, once per sweep (rare path: one atomic per entry)
__device__ __forceinline__ void hx_enqueue(const AppendArgs &a, int u)
{
    if ((uint32_t)atomicExch(&a.mark[u], (int)a.epoch) != a.epoch) {
        const int slot = atomicAdd(&a.counters[a.cout], 1);
        a.list_out[slot] = u;
    }
}

// Second phase of an append (a kernel boundary after init, so that a new node whose parent is
// also new finds that parent initialised).  Asynchronous propagation: one thread per new node carries the length of
// its own path upwards.  At every node it reaches it raises tail, level and rem, and at the top of a workflow the
// horizon; where it raises nothing it stops, since whoever left the larger values there carries them further.  Maxima
// are exact and rounding is monotone, so the fixed point is that of the level-by-level sweeps bit for bit, and no
// launch or barrier separates the levels.  Further parents that grew wait on a small stack; a walk that outgrows it or
// its step budget hands the remaining nodes to the worklist, which the sweeps after this kernel finish.
//
// What bounds it is the longest chain of memory round trips in any wavefront, and each compute unit's address unit, which
// takes one lane's scattered access at a time.  Hence first parents are known four at a time: one round trip brings four
// nodes, what they hold and the next four first parents; the raises ask for no answer, because what a walk
// carries is its own path and not what it finds (only further parents wait for theirs); and the wavefronts are spread
// over the compute units: 72 K new nodes beside a search of 23 us 40 us with a round trip of device atomics a level, each answer part
// of the next raise, and a horizon raised at every visit; so 30.  The refresh of 812 K nodes, where every node walked and raised four values,
// 157, so 44.  A walk visits 1.6 nodes on the average, but the longest in a wavefront five or six further parents, one after the
// other: where it has ended, what it needs to go on from the highest second parent comes with that one's raise, its record with the
// next four: 28 and 41 now.  The highest, as it carries the longest path: 20 graphs of 1000 nodes with up to three parents 4.9 ms, from the nearest 6.1 (5.0 where
// further parents only waited on the stack).
// (Eight first parents at a time, before that: 42 and 60, most of what they ask for lies above the point where a walk stops; two: as four.  Further parents queued in LDS for any idle lane
// of the wavefront: 30 and 59, three times the code.)
//
// REFRESH: all costs new, levels as they are.  The walks raise tails alone; rem and the horizons follow from those in a pass of
// their own.  Either every node walks, with what its tail is by now, or (leaves) only the nodes without children: their walks
// reach every other node, whose tail's mark of -1 the first to come raises.
constexpr int RELAX_STACK = 16;
constexpr int RELAX_STEPS = 1024;
// Parents beyond the second are raised this many at a time, their answers under way together.  One at a time and so: appending 50
// graphs of 8 layers of 32 nodes, all of a layer above all of the next, 6.8 and 5.6 ms; one such graph 2.1 and 1.5; 40 graphs of
// 200 nodes with up to 8 parents 3.4 and 2.8.  Four at a time take 82 registers instead of 78, a wavefront a SIMD less beside the
// search: a session of eight rounds 570 us instead of 525.
constexpr int RELAX_MANY = 3;

// block, n_blocks: the workgroup's place among those that walk (the launch may hold other workgroups too)
template <bool REFRESH>
__device__ __forceinline__ void hx_append_relax_body(const AppendArgs &a, int block, int n_blocks)
{
    // the first wavefronts of all workgroups, then the second ones
    const int lane = (int)(threadIdx.x & (HX_WAVE - 1)), wave = (int)(threadIdx.x / HX_WAVE);
    for (int i = (wave * n_blocks + block) * HX_WAVE + lane; i < a.n_new; i += n_blocks * (int)blockDim.x) {
        int stack[RELAX_STACK];
        int sp = 0, steps = 0;
        int v = a.n_old + i;
        if (REFRESH && a.leaves && a.level[v] != 0) continue;
        int4 above = a.chain[v];
        float t = 0.0f;                                      // tail and level of v as far as this walk knows
        int lv = 0;
        bool raise_rem = false;                              // rem of v is to be raised with them (else it has been)
        if (REFRESH && !a.leaves) t = __int_as_float(max(__hip_atomic_load((const int *)&a.tail[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), 0));
        for (;;) {
            const int up[HX_CHAIN] = {above.x, above.y, above.z, above.w};
            const int4 me = a.rec[v];
            int4 rec[HX_CHAIN];
            int tl[HX_CHAIN], lvl[HX_CHAIN];
#pragma unroll
            for (int k = 0; k < HX_CHAIN; ++k) {
                if (up[k] < 0) continue;
                rec[k] = a.rec[up[k]];
                tl[k] = __hip_atomic_load((const int *)&a.tail[up[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (!REFRESH) lvl[k] = __hip_atomic_load(&a.level[up[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (up[HX_CHAIN - 1] >= 0) above = a.chain[up[HX_CHAIN - 1]];
            // up the chain: source k is v or up[k - 1], its first parent up[k]
            float r = hx_node_rec_cost(me) + t;
            if (!REFRESH && raise_rem) hx_raise_max_f32(&a.rem[v], r);
            int q[HX_CHAIN];
            float src_r[HX_CHAIN];
            bool live = true, tail_up = true;
            unsigned many = 0;
#pragma unroll
            for (int k = 0; k < HX_CHAIN; ++k) {
                const int4 src = k ? rec[k ? k - 1 : 0] : me;
                q[k] = live ? src.z : -1; src_r[k] = r;
                many |= live && (src.w & HX_NODE_MANY) ? 1u << k : 0u;
                if (!REFRESH && tail_up && (src.w & HX_NODE_TOP) && src.y >= 0) hx_raise_max_f32(&a.horizon[src.y], r);
                const int u = up[k];
                live = live && u >= 0;
                tail_up = live && __float_as_int(r) > tl[k];
                const bool level_up = !REFRESH && live && lv + k + 1 > lvl[k];
                if (tail_up) atomicMax((int *)&a.tail[u], __float_as_int(r));
                if (level_up) atomicMax(&a.level[u], lv + k + 1);
                r = hx_node_rec_cost(rec[k]) + r;
                if (!REFRESH && tail_up) hx_raise_max_f32(&a.rem[u], r);
                live = tail_up || level_up;
                steps += live;
            }
            // second parents, then the others of nodes with more.  What a walk that has ended needs to go on from the highest
            // of the second parents is asked for along with the raises' answers.
            int old_t[HX_CHAIN], old_l[HX_CHAIN], pick = -1;
#pragma unroll
            for (int k = 0; k < HX_CHAIN; ++k)
                if (q[k] >= 0) {
                    old_t[k] = atomicMax((int *)&a.tail[q[k]], __float_as_int(src_r[k]));
                    if (!REFRESH) old_l[k] = atomicMax(&a.level[q[k]], lv + k + 1);
                    pick = q[k];
                }
            if (!live && pick >= 0) above = a.chain[pick];
            int next_t = -1, next_lv = 0;                    // the picked one's tail (-1: not raised) and level
            auto wait = [&](int node) {
                if (steps >= RELAX_STEPS || sp >= RELAX_STACK) hx_enqueue(a, node);
                else stack[sp++] = node;
            };
#pragma unroll
            for (int k = 0; k < HX_CHAIN; ++k)
                if (q[k] >= 0 && (__float_as_int(src_r[k]) > old_t[k] || (!REFRESH && lv + k + 1 > old_l[k]))) {
                    if (!live && steps < RELAX_STEPS && q[k] == pick) {
                        next_t = max(next_t, max(__float_as_int(src_r[k]), old_t[k]));
                        if (!REFRESH) next_lv = max(next_lv, max(lv + k + 1, old_l[k]));
                    } else wait(q[k]);
                }
            for (; many; many &= many - 1) {
                const int k = __builtin_ctz(many);
                const int s = k == 0 ? v : k == 1 ? up[0] : k == 2 ? up[1] : up[2];
                const float s_r = k == 0 ? src_r[0] : k == 1 ? src_r[1] : k == 2 ? src_r[2] : src_r[3];
                const int s_lv = lv + k;
                const int32_t *others = a.pcol + a.prow[s] + 2;
                for (int left = a.prow[s + 1] - a.prow[s] - 2; left > 0; left -= RELAX_MANY, others += RELAX_MANY) {
                    int p[RELAX_MANY], p_t[RELAX_MANY], p_l[RELAX_MANY];
#pragma unroll
                    for (int j = 0; j < RELAX_MANY; ++j) p[j] = j < left ? others[j] : -1;
#pragma unroll
                    for (int j = 0; j < RELAX_MANY; ++j)
                        if (p[j] >= 0) {
                            p_t[j] = atomicMax((int *)&a.tail[p[j]], __float_as_int(s_r));
                            if (!REFRESH) p_l[j] = atomicMax(&a.level[p[j]], s_lv + 1);
                        }
#pragma unroll
                    for (int j = 0; j < RELAX_MANY; ++j)
                        if (p[j] >= 0 && (__float_as_int(s_r) > p_t[j] || (!REFRESH && s_lv + 1 > p_l[j]))) wait(p[j]);
                }
            }
            if (live) {
                v = up[HX_CHAIN - 1];
                if (steps < RELAX_STEPS) { t = src_r[HX_CHAIN - 1]; lv += HX_CHAIN; raise_rem = false; continue; }
                hx_enqueue(a, v);
            }
            raise_rem = true;
            ++steps;
            if (next_t >= 0) {
                v = pick;
                t = __int_as_float(next_t);
                lv = next_lv;
                continue;
            }
            if (sp == 0) break;
            // a further parent, with what it holds by now
            v = stack[--sp];
            above = a.chain[v];
            t = __hip_atomic_load(&a.tail[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!REFRESH) lv = __hip_atomic_load(&a.level[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}


// An append in progress (hx_dag.hip): its first kernel has been launched, the walks and what follows them have
// not.  For the scheduling round, whose search can take the walks into its own launch.
struct HxAppendPlan {
    AppendArgs a;
    int grid;               // workgroups of 256 threads the walks would be launched with
    int n_new, n_new_edges;
};

int hx_dag_append_begin(hx_ctx *ctx, const hx_model *model, int32_t n_new, int32_t n_new_edges,
                        const int32_t *parent_row_ptr, const int32_t *parent_col_idx,
                        const int32_t *new_L_in, const int32_t *new_L_out,
                        int32_t n_types, const float *type_flops, const float *type_hbm_bw, const hx_links *links,
                        float *new_cost, const int32_t *new_wf, HxAppendPlan *plan, void *stream);
int hx_dag_append_walks(hx_ctx *ctx, const HxAppendPlan *plan, void *stream);
int hx_dag_append_end(hx_ctx *ctx, const HxAppendPlan *plan, void *stream);
