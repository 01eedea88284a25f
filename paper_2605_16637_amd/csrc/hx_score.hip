// Scoring of placement candidates: fused search
// (score + per-call argmin, no tensor written), materialised tensor, select.
//
// What is computed: Sec. 5.3 of the paper (enumerate prefill x decode
// instances, prefill finish + transfer, earliest decode finish, keep the
// earliest pair), feasibility per Sec. 5.4 Eq. (3),(4), projected ratio per
// Sec. 5.1 Eq. (2).  How it is laid out is specific to gfx950:
//
//  * The fused search does not form every pair: a candidate's cost grows with the
//    moment the KV arrives, which depends on the decode instance through its
//    class only, so the earliest arrival per class stands for all prefill
//    instances.  Lanes are calls; the pool's tables are read from LDS as
//    broadcasts (see hx_fused_search_body).
//  * Results are exactly the lexicographic minimum of (cost, p*D + d) over all
//    pairs, with the costs the materialised tensor holds, bit for bit.
#include "hx_common.hpp"
#include "hx_terms.hpp"
#include "hx_search.hpp"
#include "hx_cp.hpp"
#include "hx_append.hpp"

#include <cmath>
#include <type_traits>

namespace {

// ---- the pool as the kernels read it ---------------------------------------------

struct PrepArgs {
    HxModelF m;
    int P, D, T;
    const float *p_flops, *p_hbm;
    const int32_t *p_backlog, *p_type;
    const float *d_flops, *d_hbm;
    const int32_t *d_used, *d_cap, *d_batch, *d_qd, *d_type;
    const float *bw, *lat;
    int32_t *status;
};

// ---- common argument block of the scoring kernels ------------------------------

struct ScoreArgs {
    HxModelF m;
    int C, P, D;
    const int32_t *L_in, *L_out, *node, *wf;
    const float *elapsed, *tail, *horizon;
    int n_nodes, n_wf;
    int32_t *best_p, *best_d;
    float *best_cost, *ratio;
    float *cost;          // materialised tensor or NULL
    uint8_t *feas;        // materialised mask or NULL
    int32_t *status;
};

// projected ratio, Eq. (2), with the downstream tail of the call's node
__device__ __forceinline__ void hx_ratio(const ScoreArgs &a, int c, float best)
{
    hx_projected_ratio(a.node, a.wf, a.elapsed, a.tail, a.horizon, a.n_nodes, a.n_wf, c, best, a.status, a.ratio);
}

// ---- fused search ----------------------------------------------------------------
//
// A candidate's cost is max(done_p + x[class_p][class_d], avail_d) + dec_d.  It does not fall when its first operand
// grows, and that operand depends on the prefill instance within a class through done_p only and on the decode
// instance through its class only.  Maxima and minima round nothing and the additions are applied to the same
// operands, so the minimum over all P x D pairs is, bit for bit,
//     m[i]  = min over p of class i of done_p                      P evaluations per call
//     r[k]  = min over i of m[i] + x[i][k]                         T x T
//     best  = min over d of max(r[class_d], avail_d) + dec_d       D
// and the pair is recovered by one more pass over p: the lowest p whose candidate with the winning decode
// instance is the minimum.  P + T x T + D + P evaluations per call take the place of P x D.  Launches back to back, before
// (one wavefront per call, 2.5 instructions per pair) and now: 64 calls x 4 x 4 6.0 -> 4.2 us, 4096 x 64 x 64 7.7 -> 4.7,
// 16384 x 256 x 256 63.5 -> 8.4, 32768 x 512 x 512 450 -> 19.7, 16384 x 16 x 1024 88 -> 12.6.
//
// What bounds it: some 4 us of every launch are the chain of memory round trips (pool tables, call inputs) and the barriers
// between the passes, which is why few calls are spread over all compute units; the rest is instruction issue (a decode
// instance: 13.5 vector instructions and 2.5 LDS reads, a prefill instance: 8 + 13 and two reads in each pass; 16384 x
// 256 x 256 issues 3.4 M wave instructions, 5.5 us at one per SIMD and 4 cycles, and 0.53 M to LDS).
//
// A workgroup takes CALLS calls through the whole pool, a lane one of them; the lanes of a call in a wavefront (64 / CALLS)
// and the wavefronts deal the instances out among themselves, in turn, and read them from LDS as broadcasts.  Nothing
// is reduced across lanes but once per call and pass.
constexpr int FS_THREADS = 512;
constexpr int FS_WAVES = FS_THREADS / HX_WAVE;

// LDS carve-up shared by host (size) and device (offsets), in 4-byte words; every array starts on a 16-byte boundary
struct SearchLds {
    int P, D, calls;
    __host__ __device__ size_t pre() const { return 0; }                                   // float4 [P]: wait, 1/F, 1/B, class
    __host__ __device__ size_t dec() const { return 4 * (size_t)P; }                       // float4 [D]: wait, c1, c2, kB
    __host__ __device__ size_t dex() const { return dec() + 4 * (size_t)D; }               // int2 [D]: free tokens + 1, class
    __host__ __device__ size_t link() const { return dex() + 2 * ((size_t)(D + 1) & ~(size_t)1); }   // float2 [kT*kT]: 1/bw, latency
    __host__ __device__ size_t m() const { return link() + 2 * kT * kT; }                  // [kT][calls] earliest prefill finish per class
    __host__ __device__ size_t r() const { return m() + (size_t)kT * calls; }              // [kT][calls] earliest arrival per decode class
    __host__ __device__ size_t part() const { return r() + (size_t)kT * calls; }           // int2 [waves][calls]: cost, instance and tie of a wavefront's share
    __host__ __device__ size_t pd() const { return part() + 2 * (size_t)FS_WAVES * calls; }  // int2 [calls]: the pair
    __host__ __device__ size_t tie() const { return pd() + 2 * (size_t)calls; }            // [calls] not 0: the pair is left to hx_pair_of_tied
    __host__ __device__ size_t slot() const { return tie() + (size_t)calls; }              // [2^slot_bits()] lowest decode instance of a hash value
    __host__ __device__ int slot_bits() const { int b = 6; while ((1 << b) < 2 * D) ++b; return b; }
    __host__ __device__ size_t bytes() const { return 4 * (slot() + ((size_t)1 << slot_bits())); }
};

// the sum of a call's lengths as the capacity test takes it: it fits where need < free tokens + 1 (0: nothing fits)
__device__ __forceinline__ unsigned hx_free_plus1(int cap, int used)
{
    const long long fr = (long long)cap - (long long)used;
    return fr < 0 ? 0u : (fr > 2147483647LL ? 0x80000000u : (unsigned)fr + 1u);
}

__device__ __forceinline__ unsigned hx_alike_hash(float c1, float c2, int type, int bits)
{
    return ((__float_as_uint(c1) + (unsigned)type) * 2654435761u ^ __float_as_uint(c2) * 2246822519u) * 3266489917u >> (32 - bits);
}

// The pair of a call whose minimum `best` several decode instances attain, by one wavefront: the lowest p that
// attains it with any of them, then the lowest d that does with that p.  For a decode instance that attains it, the
// prefill instances that do so with it are those that arrive by R, the largest arrival whose candidate is still the
// minimum; R is found by bisection over the bit patterns between the earliest arrival (which attains it) and the
// minimum itself (no later arrival can), begun close to where it must be, and of a class only its largest R matters.
// (4096 calls on 64 + 64 idle instances, alike in four classes with faster links inside a class, so that this is every
// call: 9.6 us; from end to end of that range, with the call read again from memory, 11.8; pair by pair 8.8.)
// Every search carries this code, so it is kept small, its loops not unrolled: the classes one after the other instead of
// all eight side by side cost such calls 0.6 us and save every other search of a small round 0.1.
// thr: [kT] words of LDS of the wavefront's own.
__device__ __forceinline__ int2 hx_pair_of_tied(const HxCallF &cf, unsigned need, float best, int P, int D, const float4 *s_pre,
                                                const float4 *s_dec, const int2 *s_dex, const float2 *s_link, const float *r_call,
                                                int r_stride, int *thr, int lane)
{
    if (lane < kT) thr[lane] = -1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
    for (int e0 = 0; e0 < D; e0 += HX_WAVE) {
        const int e = min(e0 + lane, D - 1);
        const float4 t = s_dec[e];
        const int2 x = s_dex[e];
        const float dec = hx_decode_time(cf, t.y, t.z, t.w);
        const float r = r_call[x.y * r_stride];
        const bool hit = need < (unsigned)x.x && hx_candidate(r, t.x, dec) == best;
        int lo = __float_as_int(r), hi = hit ? __float_as_int(best) : lo;
        auto attains = [&](int arrival) { return hx_candidate(__int_as_float(arrival), t.x, dec) <= best; };
        // it is best - dec, give or take a rounding of the result: where both ends of that hold, a few steps remain of thirty
        const float about = fmaxf(best - dec, 0.0f);
        const int from = __float_as_int(about) - 2, to = __float_as_int(about + (__int_as_float(__float_as_int(best) + 1) - best)) + 2;
        if (hit && from > lo && attains(from)) lo = from;
        if (hit && to < hi && to > lo && !attains(to)) hi = to - 1;
#pragma unroll 1
        while (__builtin_amdgcn_ballot_w64(lo < hi) != 0) {
            const int mid = lo + ((hi - lo + 1) >> 1);
            const bool still = attains(mid);
            if (lo < hi) { if (still) lo = mid; else hi = mid - 1; }
        }
        if (hit) atomicMax(&thr[x.y], lo);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int R_of = thr[lane & (kT - 1)];                // lane k: of class k
    const unsigned classes = (unsigned)__builtin_amdgcn_ballot_w64(lane < kT && R_of >= 0);
    int2 out = make_int2(-1, -1);
#pragma unroll 1
    for (int p0 = 0; p0 < P; p0 += HX_WAVE) {
        const int p = min(p0 + lane, P - 1);
        const float4 t = s_pre[p];
        const float done = hx_prefill_done(cf, t.x, t.y, t.z);
        const float2 *row = s_link + __float_as_int(t.w) * kT;
        bool ok = false;
#pragma unroll 1
        for (unsigned left = classes; left; left &= left - 1) {
            const int k = __builtin_ctz(left);
            const float2 l = row[k];
            ok = ok || __float_as_int(done + hx_transfer(cf, l.x, l.y)) <= __builtin_amdgcn_readlane(R_of, k);
        }
        const unsigned long long b = __builtin_amdgcn_ballot_w64(ok && p0 + lane < P);
        if (b) { out.x = p0 + __builtin_ctzll(b); break; }
    }
    if (out.x >= 0) {
        const float4 t = s_pre[out.x];
        const float done = hx_prefill_done(cf, t.x, t.y, t.z);
        const float2 *row = s_link + __float_as_int(t.w) * kT;
    #pragma unroll 1
    for (int e0 = 0; e0 < D; e0 += HX_WAVE) {
            const int e = min(e0 + lane, D - 1);
            const float4 q = s_dec[e];
            const int2 x = s_dex[e];
            const float2 l = row[x.y];
            const float v = hx_candidate(done + hx_transfer(cf, l.x, l.y), q.x, hx_decode_time(cf, q.y, q.z, q.w));
            const unsigned long long b = __builtin_amdgcn_ballot_w64(e0 + lane < D && need < (unsigned)x.x && v == best);
            if (b) { out.y = e0 + __builtin_ctzll(b); break; }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return out;
}

// block: the workgroup's place among those that search (the launch may hold other workgroups too)
template <int CALLS>
__device__ __forceinline__ void hx_fused_search_body(const ScoreArgs &a, const PrepArgs &pa, float *smem, int block)
{
    constexpr int SUB = HX_WAVE / CALLS;                  // lanes of a wavefront that share a call
    constexpr int SLICES = SUB * FS_WAVES;
    const SearchLds lay{a.P, a.D, CALLS};
    float4 *s_pre = (float4 *)(smem + lay.pre());
    float4 *s_dec = (float4 *)(smem + lay.dec());
    int2 *s_dex = (int2 *)(smem + lay.dex());
    float2 *s_link = (float2 *)(smem + lay.link());
    float *s_m = smem + lay.m();
    float *s_r = smem + lay.r();
    int2 *s_part = (int2 *)(smem + lay.part());
    int2 *s_pd = (int2 *)(smem + lay.pd());
    int *s_tie = (int *)(smem + lay.tie());
    int *s_slot = (int *)(smem + lay.slot());
    const int slot_bits = lay.slot_bits();

    const int tid = threadIdx.x;
    const int lane = tid & (HX_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cl = lane & (CALLS - 1);                    // the lane's call within the workgroup
    const int slice = wave * SUB + lane / CALLS;
    const int base = block * CALLS;

    // what the calls say of themselves is asked for before the pool's tables; the first CALLS threads also write the
    // calls' results and ask for what the ratio needs
    const int c_in = min(base + cl, a.C - 1);
    const int L = a.L_in[c_in], O = a.L_out[c_in];
    const bool want_ratio = a.ratio != nullptr;
    const int my_c = base + tid;
    const bool mine = tid < CALLS && my_c < a.C;
    int nd = 0, w = 0;
    float el = 0.0f;
    if (mine && want_ratio) { nd = a.node[my_c]; w = a.wf[my_c]; el = a.elapsed[my_c]; }

    // ---- the pool's per-round tables, in instance order
    for (int i = tid; i < (1 << slot_bits); i += FS_THREADS) s_slot[i] = 0x7fffffff;
    {
        bool bad = false;
        const bool link_in = tid < kT * kT && tid / kT < pa.T && tid % kT < pa.T;
        const int link_at = (tid / kT) * pa.T + tid % kT;
        const float l_bw = link_in ? pa.bw[link_at] : 1.0f;
        const float l_lat = (link_in && pa.lat) ? pa.lat[link_at] : 0.0f;
        for (int i0 = 0; i0 < max(a.P, a.D); i0 += FS_THREADS) {
            const int i = i0 + tid;
            const bool hp = i < a.P, hd = i < a.D;
            const int p = hp ? i : 0, d = hd ? i : 0;
            const float pf = pa.p_flops[p], pb = pa.p_hbm[p], df = pa.d_flops[d], db = pa.d_hbm[d];
            const int bl = pa.p_backlog[p], used = pa.d_used[d], cap = pa.d_cap[d], batch = pa.d_batch[d], qd = pa.d_qd[d];
            int tp = pa.p_type[p], td = pa.d_type[d];
            if (tp < 0 || tp >= pa.T) { bad = bad || hp; tp = 0; }
            if (td < 0 || td >= pa.T) { bad = bad || hd; td = 0; }
            if (i0 == 0) __syncthreads();                          // the slots are clear; the loads above are on their way
            if (hp) {
                const float invF = 1.0f / pf;
                s_pre[p] = make_float4(hx_prefill_wait(a.m, bl, invF), invF, 1.0f / pb, __int_as_float(tp));
            }
            if (hd) {
                const HxDecF x = hx_decode_terms(a.m, used, batch, qd, 1.0f / df, 1.0f / db);
                s_dec[d] = make_float4(x.wait, x.c1, x.c2, x.kB);
                s_dex[d] = make_int2((int)hx_free_plus1(cap, used), td);
                atomicMin(&s_slot[hx_alike_hash(x.c1, x.c2, td, slot_bits)], d);
            }
        }
        if (bad) hx_raise(a.status, HX_ERR_INDEX);
        if (tid < kT * kT) s_link[tid] = make_float2(link_in ? 1.0f / l_bw : 0.0f, l_lat);
        for (int i = tid; i < kT * CALLS; i += FS_THREADS) s_m[i] = INFINITY;      // a class without instances
        if (tid < CALLS) { s_pd[tid] = make_int2(0x7fffffff, -1); s_tie[tid] = 0; }
    }
    const HxCallF cf = hx_call_terms(a.m, L, O);
    const unsigned need = (unsigned)L + (unsigned)O;      // both are >= 0: the unsigned sum cannot wrap
    __syncthreads();

    // the tail and the horizon of the ratio travel while the calls are searched
    const bool ok = nd >= 0 && nd < a.n_nodes && w >= 0 && w < a.n_wf;
    float tl = 0.0f, hz = 1.0f;
    if (mine && want_ratio && ok) { tl = a.tail[nd]; hz = a.horizon[w]; }

    // Decode instances that cannot be chosen are taken out of the search: one of the same class and per-token terms, with a
    // lower index, no later available and with no less room, is as good for every call and wins every tie.  (Idle
    // instances of a class are alike; without this nearly every call of a drained pool has several minima.)
    for (int d = tid; d < a.D; d += FS_THREADS) {
        const float4 t = s_dec[d];
        const int2 x = s_dex[d];
        const int f = s_slot[hx_alike_hash(t.y, t.z, x.y, slot_bits)];
        const float4 u = s_dec[f];
        const int2 y = s_dex[f];
        if (f < d && u.y == t.y && u.z == t.z && u.w == t.w && y.y == x.y && u.x <= t.x && (unsigned)y.x >= (unsigned)x.x) s_dex[d].x = 0;
    }
    // ---- m[i]: the earliest finish in every prefill class (finishes are not negative: their bits order like they do)
    for (int p = slice; p < a.P; p += 4 * SLICES) {
        float4 t[4];                                      // read together: none waits for the minimum before it
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = s_pre[min(p + u * SLICES, a.P - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)                       // past the end the last instance once more
            atomicMin((unsigned *)s_m + __float_as_int(t[u].w) * CALLS + cl, __float_as_uint(hx_prefill_done(cf, t[u].x, t[u].y, t[u].z)));
    }
    __syncthreads();
    // ---- r[k]: the earliest the call's KV can be at an instance of decode class k
    for (int i = tid; i < pa.T * CALLS; i += FS_THREADS) {
        const int k = i / CALLS;                          // i % CALLS is the thread's own call
        float r = INFINITY;
#pragma unroll
        for (int q = 0; q < kT; ++q) {
            const float2 l = s_link[q * kT + k];
            r = fminf(r, s_m[q * CALLS + cl] + hx_transfer(cf, l.x, l.y));      // a class without instances: +inf
        }
        s_r[k * CALLS + cl] = r;
    }
    __syncthreads();
    // ---- the minimum over the decode instances, the lowest instance that attains it, and whether others do
    float best = INFINITY;
    int bd = -1;
    bool tie = false;
#pragma unroll 8
    for (int d = slice; d < a.D; d += SLICES) {
        const float4 t = s_dec[d];
        const int2 x = s_dex[d];
        float v = hx_candidate(s_r[x.y * CALLS + cl], t.x, hx_decode_time(cf, t.y, t.z, t.w));
        v = need < (unsigned)x.x ? v : INFINITY;
        const bool lt = v < best;
        tie = !lt && (tie || v == best);
        bd = lt ? d : bd;
        best = fminf(best, v);
    }
    // instance and tie as one number: among equal costs the smallest number has the lowest instance, and there is a tie
    int key = bd * 2 + (tie ? 1 : 0);
#pragma unroll
    for (int off = CALLS; off < HX_WAVE; off <<= 1) {
        const float ov = __shfl_xor(best, off);
        const int ok2 = __shfl_xor(key, off);
        key = ov < best ? ok2 : (ov == best ? (min(key, ok2) | 1) : key);
        best = fminf(best, ov);
    }
    if (lane < CALLS) s_part[wave * CALLS + cl] = make_int2(__float_as_int(best), key);
    __syncthreads();
    {
        int2 q[FS_WAVES];
#pragma unroll
        for (int v = 0; v < FS_WAVES; ++v) q[v] = s_part[v * CALLS + cl];
        best = __int_as_float(q[0].x);
        key = q[0].y;
#pragma unroll
        for (int v = 1; v < FS_WAVES; ++v) {
            const float ov = __int_as_float(q[v].x);
            key = ov < best ? q[v].y : (ov == best ? (min(key, q[v].y) | 1) : key);
            best = fminf(best, ov);
        }
    }
    const bool any = best < INFINITY;
    const int d_win = any ? key >> 1 : 0;
    const float4 t_win = s_dec[d_win];
    const int k_win = s_dex[d_win].y;
    const float dec_win = hx_decode_time(cf, t_win.y, t_win.z, t_win.w);
    if (slice == 0 && any) s_pd[cl].y = d_win;
    // Several decode instances attain a minimum.  Those of the winner's class, or of one with the same links to it, and with
    // its decode time do so with the same prefill instances as the winner, whatever their availability: nothing
    // changes, the lowest instance has been kept.  (Classes with the same links: 4096 calls on an idle pool of 64 + 64
    // alike instances in four classes 11.4 -> 6.8 us.)  A call that has others (rare) is left to hx_pair_of_tied.
    // (Every wavefront sees every call: uniform.)
    const bool tied = __builtin_amdgcn_ballot_w64(any && (key & 1)) != 0;
    if (tied) {
#pragma unroll 1
        for (int d = slice; d < a.D; d += SLICES) {
            const float4 t = s_dec[d];
            const int2 x = s_dex[d];
            const float dec = hx_decode_time(cf, t.y, t.z, t.w);
            if (any && need < (unsigned)x.x && (x.y != k_win || dec != dec_win) &&
                hx_candidate(s_r[x.y * CALLS + cl], t.x, dec) == best) {
                bool alike = dec == dec_win;
#pragma unroll 1
                for (int q = 0; q < pa.T; ++q) {
                    const float2 u = s_link[q * kT + x.y], v = s_link[q * kT + k_win];
                    alike = alike && u.x == v.x && u.y == v.y;
                }
                if (!alike) s_tie[cl] = 1;
            }
        }
    }
    // ---- the lowest prefill instance that attains the minimum with the winner
    int p_low = 0x7fffffff;
#pragma unroll 8
    for (int p = slice; p < a.P; p += SLICES) {
        const float4 t = s_pre[p];
        const float2 l = s_link[__float_as_int(t.w) * kT + k_win];
        const float v = hx_candidate(hx_prefill_done(cf, t.x, t.y, t.z) + hx_transfer(cf, l.x, l.y), t_win.x, dec_win);
        if (v == best) p_low = min(p_low, p);
    }
#pragma unroll
    for (int off = CALLS; off < HX_WAVE; off <<= 1) p_low = min(p_low, __shfl_xor(p_low, off));
    if (lane < CALLS && any && p_low < 0x7fffffff) atomicMin(&s_pd[cl].x, p_low);
    __syncthreads();
    if (tied) {
#pragma unroll 1
        for (int ct = wave; ct < CALLS; ct += FS_WAVES) {
            if (s_tie[ct] == 0) continue;
            const int Lt = __builtin_amdgcn_readlane(L, ct), Ot = __builtin_amdgcn_readlane(O, ct);      // lane ct's call is call ct
            const float b = hx_lane_value(best, ct);
            // its words of LDS: the class minima, which nobody reads any more
            const int2 pd = hx_pair_of_tied(hx_call_terms(a.m, Lt, Ot), (unsigned)Lt + (unsigned)Ot, b, a.P, a.D, s_pre, s_dec, s_dex, s_link,
                                            s_r + ct, CALLS, (int *)s_m + wave * kT, lane);
            if (lane == 0) s_pd[ct] = pd;
        }
        __syncthreads();
    }
    if (mine) {                                           // the thread's own call is call my_c
        const int2 pd = s_pd[tid];
        const bool placed = any && pd.x != 0x7fffffff;
        a.best_p[my_c] = placed ? pd.x : -1;
        a.best_d[my_c] = placed ? pd.y : -1;
        a.best_cost[my_c] = best;
        if (want_ratio) {
            if (!ok) hx_raise(a.status, HX_ERR_INDEX);
            hx_store_bits(a.ratio, my_c, hx_ratio_bits(el, best, tl, hz, ok));      // Eq. (2), as hx_projected_ratio forms it
        }
    }
}

template <int CALLS>
__global__ __launch_bounds__(FS_THREADS) void hx_fused_search_kernel(ScoreArgs a, PrepArgs pa)
{
    extern __shared__ __align__(16) float smem[];
    hx_fused_search_body<CALLS>(a, pa, smem, (int)blockIdx.x);
}

// ---- the first kernel of a scheduling round that brings its whole graph: reveal and search in one launch ----
//
// The horizon refresh (node cost + critical path, what hx_cp_cost_kernel does) and the search do not depend on each
// other -- only the ratio needs both, and it is formed by the commit kernel that follows -- so they share a launch:
// the first n_reveal workgroups take workflows exactly as hx_cp_cost_kernel's do (same bodies, a node per lane or thread, the
// cost's decode classes one after the other to stay within the search's registers), the others search.  Same
// results as the two kernels, one launch and the gap before it less: both halves are chains of memory round trips,
// which run side by side.  The reveal's chain is the longer one, so its workgroups come first.  Six wavefronts a SIMD, so that
// three workgroups are on a compute unit: 16384 calls on 256 + 256 with 82000 nodes 14.6 -> 12.5 us (85 registers, two workgroups: 16.1).
constexpr int RV_NMAX = 512;             // nodes staged per run of a reveal workgroup

struct RevealLds {
    union {
        CpNode node[RV_NMAX + 1];
        CpWave wave[FS_WAVES];
    };
    CostTables tab;
    int any;
};

template <int CALLS>
__global__ __launch_bounds__(FS_THREADS, 6) void hx_reveal_search_kernel(ScoreArgs a, PrepArgs pa, CpArgs cp, NodeCostArgs nc, int wpb,
                                                                      int wpv, int n_reveal)
{
    extern __shared__ __align__(16) float smem[];
    if ((int)blockIdx.x < n_reveal) {
        RevealLds *l = (RevealLds *)smem;
        if (wpv && hx_cp_waves_body<FS_THREADS>(cp, wpb, wpv, l->wave, nc, l->tab, (int)blockIdx.x)) return;
        hx_cp_local_body<RV_NMAX, true, false, FS_THREADS>(cp, wpb, l->node, l->any, &nc, &l->tab, (int)blockIdx.x, wpv != 0);
        return;
    }
    hx_fused_search_body<CALLS>(a, pa, smem, (int)blockIdx.x - n_reveal);
}

// The same for a round that appends to the context's graph: the append's walks (hx_append_relax_kernel's work: one
// thread per new node, a chain of device-scope atomics up its ancestors) take the first n_lead workgroups of the
// search's launch.  They are all latency and no arithmetic, and longer than the search that runs beside them.
template <int CALLS>
__global__ __launch_bounds__(FS_THREADS) void hx_relax_search_kernel(ScoreArgs a, PrepArgs pa, AppendArgs ap, int n_lead)
{
    extern __shared__ __align__(16) float smem[];
    if ((int)blockIdx.x < n_lead) {
        hx_append_relax_body<false>(ap, (int)blockIdx.x, n_lead);
        return;
    }
    hx_fused_search_body<CALLS>(a, pa, smem, (int)blockIdx.x - n_lead);
}

// ---- materialised tensor ------------------------------------------------------------

// A workgroup takes nc calls at a time (nc = 4 on small pools, where one call's share of the tensor is a few
// KB and the barriers and the per-call tables would otherwise cost as much as the stores; 1 on large ones).
// LDS: per call of the batch the prefill finish per instance, the decode time per instance and the class-pair
// transfer times, each worked out by 256 / nc threads; beside them what does not depend on the call (waits,
// per-token terms, classes), which every workgroup derives for itself from the pool, under the first call's lengths: as a
// kernel of one workgroup before this one they took 3.5 us (4096 x 64 x 64 with the selection after it 38.8 -> 36.1).
// Bound: the stores (a plain fill of 4096 x 64 x 64 takes 12.3 us), and before the first of them one memory round trip and the tables'
// divisions, in which no workgroup writes: everything is asked for together (4096 x 64 x 64 15.5 -> 14.6 us, 64 x 8 x 8 4.1 -> 3.7; prefill
// instances, decode instances, links and calls one after the other before).
__global__ __launch_bounds__(256) void hx_materialise_kernel(ScoreArgs a, PrepArgs t, int nc)
{
    extern __shared__ __align__(16) float smem[];
    const int P4 = (a.P + 3) & ~3, D4 = (a.D + 3) & ~3;      // every array starts on a 16-byte boundary
    float *s_done = smem;                       // [nc][P4] per call
    float *s_dec = s_done + nc * P4;            // [nc][D4] per call
    float *s_x = s_dec + nc * D4;               // [nc][kT*kT] per call
    float *s_wait = s_x + nc * kT * kT;         // [D]
    int *s_ptype = (int *)(s_wait + D4);        // [P]
    int *s_dtype = s_ptype + P4;                // [D]
    float *s_pw = (float *)(s_dtype + D4);      // [P] prefill wait, 1/F, 1/B
    float *s_pF = s_pw + P4;
    float *s_pB = s_pF + P4;
    float *s_c1 = s_pB + P4;                    // [D] decode per-token terms and free tokens, by instance
    float *s_c2 = s_c1 + D4;
    float *s_kB = s_c2 + D4;
    int *s_free = (int *)(s_kB + D4);
    float *s_lbw = (float *)(s_free + D4);      // [kT*kT] link tables
    float *s_llat = s_lbw + kT * kT;
    const int tid = threadIdx.x;
    // rows of the tensor are 16-byte aligned and a whole number of quads long
    const bool vec4 = (a.D & 3) == 0 && a.D >= 4 && (reinterpret_cast<uintptr_t>(a.cost) & 15) == 0;
    // the part of the workgroup that works out the tables of one call of the batch
    const int per_call = blockDim.x / nc;
    const int slot = tid / per_call, tq = tid - slot * per_call;
    // everything is asked for before the first of it is used: the first calls' lengths, the links, an instance of either side a thread
    const int c_first = min((int)(blockIdx.x * nc) + slot, a.C - 1);
    int L = a.L_in[c_first], O = a.L_out[c_first];
    const bool link_in = tid < kT * kT && tid / kT < t.T && tid % kT < t.T;
    const int link_at = (tid / kT) * t.T + tid % kT;
    const float l_bw = link_in ? t.bw[link_at] : 1.0f;
    const float l_lat = link_in && t.lat ? t.lat[link_at] : 0.0f;
    for (int i0 = 0; i0 < max(a.P, a.D); i0 += (int)blockDim.x) {
        const int i = i0 + tid;
        const bool hp = i < a.P, hd = i < a.D;
        const int p = hp ? i : 0, d = hd ? i : 0;
        const float pf = t.p_flops[p], pb = t.p_hbm[p], df = t.d_flops[d], db = t.d_hbm[d];
        const int bl = t.p_backlog[p], used = t.d_used[d], cap = t.d_cap[d], batch = t.d_batch[d], qd = t.d_qd[d];
        int kp = t.p_type[p], kd = t.d_type[d];
        if (kp < 0 || kp >= t.T) { if (hp) hx_raise(a.status, HX_ERR_INDEX); kp = 0; }
        if (kd < 0 || kd >= t.T) { if (hd) hx_raise(a.status, HX_ERR_INDEX); kd = 0; }
        if (hp) {
            const float invF = 1.0f / pf;
            s_pw[p] = hx_prefill_wait(a.m, bl, invF); s_pF[p] = invF; s_pB[p] = 1.0f / pb; s_ptype[p] = kp;
        }
        if (hd) {
            const HxDecF x = hx_decode_terms(a.m, used, batch, qd, 1.0f / df, 1.0f / db);
            const long long fr = (long long)cap - (long long)used;
            s_c1[d] = x.c1; s_c2[d] = x.c2; s_kB[d] = x.kB; s_wait[d] = x.wait; s_dtype[d] = kd;
            s_free[d] = fr < -1 ? -1 : (fr > 2147483647LL ? 2147483647 : (int)fr);
        }
    }
    if (tid < kT * kT) { s_lbw[tid] = link_in ? 1.0f / l_bw : 0.0f; s_llat[tid] = l_lat; }
    for (int c0 = blockIdx.x * nc; c0 < a.C; c0 += gridDim.x * nc) {
        const int cs = c0 + slot;
        const bool live = cs < a.C;
        const HxCallF cf = hx_call_terms(a.m, L, O);
        const int L_now = L, O_now = O;
        if (c0 + (int)(gridDim.x * nc) < a.C) {            // the next calls' lengths
            const int c_next = min(cs + (int)(gridDim.x * nc), a.C - 1);
            L = a.L_in[c_next]; O = a.L_out[c_next];
        }
        __syncthreads();
        if (live) {
            for (int p = tq; p < a.P; p += per_call) s_done[slot * P4 + p] = hx_prefill_done(cf, s_pw[p], s_pF[p], s_pB[p]);
            for (int d = tq; d < a.D; d += per_call) {
                const bool fits = hx_fits(L_now, O_now, s_free[d]);
                s_dec[slot * D4 + d] = fits ? hx_decode_time(cf, s_c1[d], s_c2[d], s_kB[d]) : INFINITY;
                if (a.feas) a.feas[(size_t)cs * a.D + d] = fits ? 1 : 0;
            }
            for (int i = tq; i < kT * kT; i += per_call) s_x[slot * kT * kT + i] = hx_transfer(cf, s_lbw[i], s_llat[i]);
        }
        __syncthreads();
        if (a.cost) {
            const int n_here = min(nc, a.C - c0);
            for (int s = 0; s < n_here; ++s) {
                float *out = a.cost + (size_t)(c0 + s) * a.P * a.D;
                const float *done_s = s_done + s * P4, *dec_s = s_dec + s * D4, *x_s = s_x + s * kT * kT;
                // (p, d) of the elements a thread writes advance without a division: by blockDim positions at a time
                if (vec4) {
                    // four neighbouring decode instances per step, one 16-byte store
                    const int dq = a.D >> 2;
                    const int step_p = blockDim.x / dq, step_q = blockDim.x % dq;
                    int p = tid / dq, q = tid - p * dq;
                    for (; p < a.P; p += step_p) {
                        const float done = done_s[p];
                        const float *xr = x_s + s_ptype[p] * kT;
                        const float4 w = reinterpret_cast<const float4 *>(s_wait)[q];
                        const float4 tm = reinterpret_cast<const float4 *>(dec_s)[q];
                        const int4 k = reinterpret_cast<const int4 *>(s_dtype)[q];
                        float4 v;
                        v.x = hx_candidate(done + xr[k.x], w.x, tm.x);
                        v.y = hx_candidate(done + xr[k.y], w.y, tm.y);
                        v.z = hx_candidate(done + xr[k.z], w.z, tm.z);
                        v.w = hx_candidate(done + xr[k.w], w.w, tm.w);
                        reinterpret_cast<float4 *>(out + (size_t)p * a.D)[q] = v;
                        q += step_q;
                        if (q >= dq) { q -= dq; ++p; }
                    }
                } else {
                    const int step_p = blockDim.x / a.D, step_d = blockDim.x % a.D;
                    int p = tid / a.D, d = tid - p * a.D;
                    for (; p < a.P; p += step_p) {
                        out[(size_t)p * a.D + d] = hx_candidate(done_s[p] + x_s[s_ptype[p] * kT + s_dtype[d]], s_wait[d], dec_s[d]);
                        d += step_d;
                        if (d >= a.D) { d -= a.D; ++p; }
                    }
                }
            }
        }
    }
}
// Up to SELECT_WAVE pairs in whole quads: a wavefront takes a call, U 16-byte loads of it in flight per lane, and reduces it
// without a barrier; the workgroup per call below spends most of a short row on its reduction.  Launches back to back (us), workgroup
// and wavefront, U = 1 up to a quad a lane, else 8: 16384 calls x 8 x 8 15.7 and 4.3, 4096 x 16 x 16 6.0 and 2.7, 64 x 4 x 4 3.1 and 2.4,
// 64 x 64 x 64 3.5 and 2.9, 4096 x 64 x 64 12.8 and 11.8 (67 MB at 5.7 TB/s, more than a copy from memory reaches: just written, they lie in the
// last-level cache).  (U = 8 for short rows too: the same quad eight times, 7.5 us for 16384 x 8 x 8, and 3.2 for 64 x 4 x 4, rows that share a
// cache line.)  Longer rows are more turns of one wavefront, a chain of memory round trips that the workgroup splits: 64 calls x 80 x 100 4.0
// and 3.7, 96 x 128 4.3 and 4.5, 256 x 128 6.3 and 8.5; 1024 calls x 65 x 64 4.2 and 4.4, x 80 x 100 6.7 and 6.0, x 128 x 128 12.6 and
// 12.1; 4096 x 128 x 128 41 and 43.  At 4096 pairs the wavefront wins for any number of calls, at twice that within 11 % either way.
constexpr int SELECT_WAVE = 4096;
template <int U>
__global__ __launch_bounds__(256) void hx_select_wave_kernel(ScoreArgs a)
{
    const int lane = threadIdx.x & (HX_WAVE - 1);
    const unsigned wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x / HX_WAVE) + threadIdx.x / HX_WAVE));
    const int n4 = (a.P * a.D) >> 2;
    for (unsigned c = wave; c < (unsigned)a.C; c += gridDim.x * (blockDim.x / HX_WAVE)) {       // (may step past 2^31)
        const float4 *row = reinterpret_cast<const float4 *>(a.cost + (size_t)c * ((size_t)n4 * 4));
        float bv = INFINITY;
        int bi = 0x7fffffff;
        for (int i0 = lane; i0 < n4; i0 += U * HX_WAVE) {
            float4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = row[min(i0 + u * HX_WAVE, n4 - 1)];       // (past the end the last quad once more)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = min(i0 + u * HX_WAVE, n4 - 1) << 2;
                if (x[u].x < bv) { bv = x[u].x; bi = i; }
                if (x[u].y < bv) { bv = x[u].y; bi = i + 1; }
                if (x[u].z < bv) { bv = x[u].z; bi = i + 2; }
                if (x[u].w < bv) { bv = x[u].w; bi = i + 3; }
            }
        }
        const float best = hx_wave_min(bv);
        bi = hx_wave_min(bv == best ? bi : 0x7fffffff);
        if (lane == 0) {
            const bool any = best < INFINITY;
            a.best_p[c] = any ? bi / a.D : -1;
            a.best_d[c] = any ? bi % a.D : -1;
            a.best_cost[c] = best;
            if (a.ratio) hx_ratio(a, c, best);
        }
    }
}

__global__ __launch_bounds__(256) void hx_select_kernel(ScoreArgs a)
{
    __shared__ float s_v[4];
    __shared__ int s_i[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = a.P * a.D;
    const bool vec4 = (n & 3) == 0 && (reinterpret_cast<uintptr_t>(a.cost) & 15) == 0;
    for (unsigned c = blockIdx.x; c < (unsigned)a.C; c += gridDim.x) {
        const float *row = a.cost + (size_t)c * n;
        float bv = INFINITY;
        int bi = 0x7fffffff;
        if (vec4) {
            // 16-byte loads, two in flight per thread; indices grow within a quad and from quad to quad
            const float4 *row4 = reinterpret_cast<const float4 *>(row);
            const int n4 = n >> 2;
            int i4 = tid;
            for (; i4 + (int)blockDim.x < n4; i4 += 2 * blockDim.x) {
                const float4 x = row4[i4], y = row4[i4 + blockDim.x];
                const int i = i4 << 2, j = (i4 + blockDim.x) << 2;
                if (x.x < bv) { bv = x.x; bi = i; }
                if (x.y < bv) { bv = x.y; bi = i + 1; }
                if (x.z < bv) { bv = x.z; bi = i + 2; }
                if (x.w < bv) { bv = x.w; bi = i + 3; }
                if (y.x < bv) { bv = y.x; bi = j; }
                if (y.y < bv) { bv = y.y; bi = j + 1; }
                if (y.z < bv) { bv = y.z; bi = j + 2; }
                if (y.w < bv) { bv = y.w; bi = j + 3; }
            }
            if (i4 < n4) {
                const float4 x = row4[i4];
                const int i = i4 << 2;
                if (x.x < bv) { bv = x.x; bi = i; }
                if (x.y < bv) { bv = x.y; bi = i + 1; }
                if (x.z < bv) { bv = x.z; bi = i + 2; }
                if (x.w < bv) { bv = x.w; bi = i + 3; }
            }
        } else {
            for (int i = tid; i < n; i += blockDim.x) {     // i grows: "<" keeps the lowest index of this thread
                float v = row[i];
                if (v < bv) { bv = v; bi = i; }
            }
        }
#pragma unroll
        for (int off = HX_WAVE / 2; off > 0; off >>= 1) {
            float ov = __shfl_xor(bv, off);
            int oi = __shfl_xor(bi, off);
            bool take = ov < bv || (ov == bv && oi < bi);
            bv = take ? ov : bv;
            bi = take ? oi : bi;
        }
        __syncthreads();
        if (lane == 0) { s_v[wave] = bv; s_i[wave] = bi; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
                if (s_v[w] < bv || (s_v[w] == bv && s_i[w] < bi)) { bv = s_v[w]; bi = s_i[w]; }
            bool any = bv < INFINITY;
            a.best_p[c] = any ? bi / a.D : -1;
            a.best_d[c] = any ? bi % a.D : -1;
            a.best_cost[c] = bv;
            if (a.ratio) hx_ratio(a, c, bv);
        }
    }
}

// the urgency fold on its own: Eq. (2) from best costs found earlier
__global__ __launch_bounds__(256) void hx_urgency_kernel(const int32_t *node, const int32_t *wf, const float *elapsed,
                                                         const float *best_cost, const float *tail, const float *horizon,
                                                         int n_nodes, int n_wf, int C, float *ratio, int32_t *status)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < C) hx_projected_ratio(node, wf, elapsed, tail, horizon, n_nodes, n_wf, c, best_cost[c], status, ratio);
}

// fused outputs when the pool is empty: nothing is feasible
__global__ void hx_no_pool_kernel(ScoreArgs a)
{
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.C) return;
    a.best_p[c] = -1; a.best_d[c] = -1; a.best_cost[c] = INFINITY;
    if (a.ratio) hx_ratio(a, c, INFINITY);
}

HxModelF to_model(const hx_model *m)
{
    return HxModelF{m->kv_bytes_per_token, m->flops_per_token, m->attn_flops_per_token2,
                    m->weight_bytes, m->nominal_batch};
}

// the pool tables as the table derivation reads them (pointers checked by the caller)
PrepArgs make_prep_args(hx_ctx *ctx, const hx_model *model, const hx_prefill_tab *pre, const hx_decode_tab *dec,
                        const hx_links *links)
{
    PrepArgs pa{};
    pa.m = to_model(model); pa.P = pre->n; pa.D = dec->n; pa.T = links->n_types;
    pa.p_flops = pre->flops; pa.p_hbm = pre->hbm_bw; pa.p_backlog = pre->backlog_tok; pa.p_type = pre->type;
    pa.d_flops = dec->flops; pa.d_hbm = dec->hbm_bw; pa.d_used = dec->used_tok; pa.d_cap = dec->cap_tok;
    pa.d_batch = dec->batch; pa.d_qd = dec->qd_tok; pa.d_type = dec->type;
    pa.bw = links->bw; pa.lat = links->latency; pa.status = ctx->d_status;
    return pa;
}

int check_ratio_inputs(hx_ctx *ctx, const hx_calls *calls, const float *tail, const float *horizon,
                       int32_t n_nodes, int32_t n_wf, const float *ratio)
{
    if (!ratio) return HX_OK;
    HX_REQUIRE(ctx, calls && calls->node && calls->wf && calls->elapsed && tail && horizon,
               HX_ERR_INVALID_ARG, "ratio needs calls.node, calls.wf, calls.elapsed, tail and horizon");
    HX_REQUIRE(ctx, n_nodes >= 0 && n_wf >= 0, HX_ERR_INVALID_ARG, "negative n_nodes or n_wf");
    return HX_OK;
}

}  // namespace

// Validates the pool tables.
int hx_check_pool(hx_ctx *ctx, const hx_model *model, const hx_prefill_tab *pre, const hx_decode_tab *dec, const hx_links *links)
{
    HX_REQUIRE(ctx, model && pre && dec && links, HX_ERR_INVALID_ARG, "NULL table");
    const int P = pre->n, D = dec->n, T = links->n_types;
    HX_REQUIRE(ctx, P >= 0 && D >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, T >= 1 && T <= HX_MAX_TYPES, HX_ERR_SHAPE, "n_types %d outside 1..%d", T, HX_MAX_TYPES);
    HX_REQUIRE(ctx, P <= HX_MAX_INSTANCES && D <= HX_MAX_INSTANCES, HX_ERR_SHAPE,
               "pool %d x %d beyond %d instances per side", P, D, HX_MAX_INSTANCES);
    HX_REQUIRE(ctx, P == 0 || (pre->flops && pre->hbm_bw && pre->backlog_tok && pre->type),
               HX_ERR_INVALID_ARG, "NULL member in prefill table");
    HX_REQUIRE(ctx, D == 0 || (dec->flops && dec->hbm_bw && dec->used_tok && dec->cap_tok && dec->batch &&
                               dec->qd_tok && dec->type), HX_ERR_INVALID_ARG, "NULL member in decode table");
    HX_REQUIRE(ctx, links->bw, HX_ERR_INVALID_ARG, "links.bw is NULL");
    return HX_OK;
}

namespace {

// reveal: NULL, or the horizon refresh of the same round (hx_horizons_plan), to ride in the search's launch if the
// round is small enough for that: *revealed says whether it did.  walks: NULL, or an append of the same round that
// has begun (hx_dag_append_begin), whose walks are to ride in the search's launch likewise.  With a reveal the ratio is only checked, not
// written -- the horizons are not there yet; the caller forms it afterwards -- and nothing but the fused search is
// launched: if the reveal does not fit, nothing at all is, and the caller makes the calls one after the other.
int score_placements(hx_ctx *ctx, const hx_model *model, const hx_calls *calls,
                     const hx_prefill_tab *pre, const hx_decode_tab *dec, const hx_links *links,
                     const float *tail, const float *horizon, int32_t n_nodes, int32_t n_wf,
                     float *cost, uint8_t *feas,
                     int32_t *best_p, int32_t *best_d, float *best_cost, float *ratio,
                     const HxHorizonsPlan *reveal, const HxAppendPlan *walks, bool *revealed, void *stream_)
{
    HX_REQUIRE(ctx, model && calls && pre && dec && links, HX_ERR_INVALID_ARG, "NULL table");
    const int C = calls->n, P = pre->n, D = dec->n, T = links->n_types;
    HX_REQUIRE(ctx, C >= 0 && P >= 0 && D >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, T >= 1 && T <= HX_MAX_TYPES, HX_ERR_SHAPE, "n_types %d outside 1..%d", T, HX_MAX_TYPES);
    HX_REQUIRE(ctx, P <= HX_MAX_INSTANCES && D <= HX_MAX_INSTANCES, HX_ERR_SHAPE,
               "pool %d x %d beyond %d instances per side", P, D, HX_MAX_INSTANCES);
    const bool fused = best_p || best_d || best_cost;
    HX_REQUIRE(ctx, !fused || (best_p && best_d && best_cost), HX_ERR_INVALID_ARG,
               "best_p, best_d, best_cost must be given together");
    HX_REQUIRE(ctx, fused || cost || feas, HX_ERR_INVALID_ARG, "no output requested");
    HX_REQUIRE(ctx, !ratio || fused, HX_ERR_INVALID_ARG, "ratio needs the fused outputs");
    HX_REQUIRE(ctx, C == 0 || (calls->L_in && calls->L_out), HX_ERR_INVALID_ARG, "calls.L_in / L_out is NULL");
    HX_REQUIRE(ctx, P == 0 || (pre->flops && pre->hbm_bw && pre->backlog_tok && pre->type),
               HX_ERR_INVALID_ARG, "NULL member in prefill table");
    HX_REQUIRE(ctx, D == 0 || (dec->flops && dec->hbm_bw && dec->used_tok && dec->cap_tok && dec->batch &&
                               dec->qd_tok && dec->type), HX_ERR_INVALID_ARG, "NULL member in decode table");
    HX_REQUIRE(ctx, links->bw, HX_ERR_INVALID_ARG, "links.bw is NULL");
    HX_REQUIRE(ctx, !cost || (double)C * P * D < 9.0e18, HX_ERR_SHAPE, "tensor too large");
    HX_REQUIRE(ctx, (long long)P * D <= 2147483647LL, HX_ERR_SHAPE, "P*D beyond int32");
    if (int rc = check_ratio_inputs(ctx, calls, tail, horizon, n_nodes, n_wf, ratio)) return rc;
    if (C == 0) return HX_OK;

    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;

    ScoreArgs a{};
    a.m = to_model(model);
    a.C = C; a.P = P; a.D = D;
    a.L_in = calls->L_in; a.L_out = calls->L_out; a.node = calls->node; a.wf = calls->wf;
    a.elapsed = calls->elapsed; a.tail = tail; a.horizon = horizon; a.n_nodes = n_nodes; a.n_wf = n_wf;
    a.best_p = best_p; a.best_d = best_d; a.best_cost = best_cost; a.ratio = (reveal || walks) ? nullptr : ratio;
    a.cost = cost; a.feas = feas; a.status = ctx->d_status;

    if (reveal && (P == 0 || D == 0 || !fused || cost || feas || reveal->grid == 0)) return HX_OK;      // not this way
    if (walks && (P == 0 || D == 0 || !fused || cost || feas || walks->grid == 0)) return HX_OK;
    if (P == 0 || D == 0) {
        if (fused) {
            hx_no_pool_kernel<<<(C + 255) / 256, 256, 0, stream>>>(a);
            return hx_check_launch(ctx, "hx_no_pool_kernel");
        }
        return HX_OK;
    }

    if (fused) {
        // the search derives the per-round tables of the pool in its own workgroups: no launch of its own for them
        const PrepArgs pa = make_prep_args(ctx, model, pre, dec, links);
        // Calls per workgroup: as few as spread the calls over every compute unit (the tables are derived once per
        // workgroup, in the same time however many calls follow), 64 at most.  Two workgroups to a compute unit
        // beat one of twice the calls as long as the tables are short beside the passes (16384 x 256 x 256: 8.4 us with 32
        // calls each, 9.4 with 64); from 65 calls per compute unit on there are two of 64 (32768 x 512 x 512: 19.7 us,
        // 21.7 with 32; 65536 x 256 x 256: 19.7, 23.6 with 32).  8192 x 64 x 64 takes 4.9 us with 32 and 5.3 with 16.
        const int per_cu = (C + ctx->num_cu - 1) / ctx->num_cu;
        const int calls_per_wg = per_cu > 64 ? 64 : per_cu > 16 ? 32 : per_cu > 8 ? 16 : 8;
        const int n_search = (C + calls_per_wg - 1) / calls_per_wg;
        const size_t lds = SearchLds{P, D, calls_per_wg}.bytes();
        auto by_calls = [&](auto &&launch) {
            if (calls_per_wg == 64) launch(std::integral_constant<int, 64>{});
            else if (calls_per_wg == 32) launch(std::integral_constant<int, 32>{});
            else if (calls_per_wg == 16) launch(std::integral_constant<int, 16>{});
            else launch(std::integral_constant<int, 8>{});
        };
        if (reveal) {
            // not this way if the reveal's units are too large for its staging area
            const long long nodes_per_unit = (long long)reveal->a.n_nodes * reveal->wpb / (reveal->a.n_wf > 0 ? reveal->a.n_wf : 1);
            if (nodes_per_unit > RV_NMAX * 7 / 10) return HX_OK;
            // wavefronts of a workgroup that take workflows: no more than give every compute unit a workgroup, so that one that takes its
            // workflows as a slice after all has few (1023 workflows of 24 to 70 nodes 18.4 us a round with eight, 16.6 with four; of 10 to 30 12.0 and 11.5)
            const int fill = reveal->wpv ? (reveal->a.n_wf + reveal->wpv * ctx->num_cu - 1) / (reveal->wpv * ctx->num_cu) : 0;
            const int wpb = reveal->wpv ? reveal->wpv * (fill < FS_WAVES ? fill : FS_WAVES) : reveal->wpb, n_reveal = (reveal->a.n_wf + wpb - 1) / wpb;
            const size_t lds_both = lds > sizeof(RevealLds) ? lds : sizeof(RevealLds);
            by_calls([&](auto calls) {
                hx_reveal_search_kernel<calls()><<<n_reveal + n_search, FS_THREADS, lds_both, stream>>>(
                    a, pa, reveal->a, reveal->nc, wpb, reveal->wpv, n_reveal);
            });
            if (int rc = hx_check_launch(ctx, "hx_reveal_search_kernel")) return rc;
            *revealed = true;
            return HX_OK;
        }
        if (walks) {
            // a workgroup of walks to every compute unit, as far as there are wavefronts of them
            const int most = (walks->a.n_new + HX_WAVE - 1) / HX_WAVE, least = (walks->a.n_new + FS_THREADS - 1) / FS_THREADS;
            const int n_lead = least > ctx->num_cu ? least : (most < ctx->num_cu ? most : ctx->num_cu);
            by_calls([&](auto calls) {
                hx_relax_search_kernel<calls()><<<n_lead + n_search, FS_THREADS, lds, stream>>>(a, pa, walks->a, n_lead);
            });
            if (int rc = hx_check_launch(ctx, "hx_relax_search_kernel")) return rc;
            *revealed = true;
            return HX_OK;
        }
        by_calls([&](auto calls) { hx_fused_search_kernel<calls()><<<n_search, FS_THREADS, lds, stream>>>(a, pa); });
        if (int rc = hx_check_launch(ctx, "hx_fused_search_kernel")) return rc;
    }
    if (cost || feas) {
        if (int rc = hx_check_pool(ctx, model, pre, dec, links)) return rc;
        const int P4 = (P + 3) & ~3, D4 = (D + 3) & ~3;
        const int nc = (long long)P * D <= 16384 && C >= 4 * ctx->num_cu * 4 ? 4 : 1;      // calls per workgroup at a time
        const size_t lds = 4 * ((size_t)nc * (P4 + D4 + kT * kT) + 4 * P4 + 6 * D4 + 2 * kT * kT);
        const int batches = (C + nc - 1) / nc;
        const int grid = batches < ctx->num_cu * 8 ? batches : ctx->num_cu * 8;
        hx_materialise_kernel<<<grid, 256, lds, stream>>>(a, make_prep_args(ctx, model, pre, dec, links), nc);
        if (int rc = hx_check_launch(ctx, "hx_materialise_kernel")) return rc;
    }
    return HX_OK;
}

}  // namespace

extern "C" int hx_score_placements(hx_ctx *ctx, const hx_model *model, const hx_calls *calls,
                                   const hx_prefill_tab *pre, const hx_decode_tab *dec,
                                   const hx_links *links,
                                   const float *tail, const float *horizon, int32_t n_nodes, int32_t n_wf,
                                   float *cost, uint8_t *feas,
                                   int32_t *best_p, int32_t *best_d, float *best_cost, float *ratio,
                                   void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    return score_placements(ctx, model, calls, pre, dec, links, tail, horizon, n_nodes, n_wf, cost, feas,
                            best_p, best_d, best_cost, ratio, nullptr, nullptr, nullptr, stream_);
}

// The horizon refresh `reveal` and hx_score_placements (fused outputs) in one launch, where the round is small
// enough (*revealed; otherwise nothing has been launched).  ratio is checked like hx_score_placements' but not
// written: the caller forms it once the launch has produced the horizons (the commit kernel does).
int hx_reveal_search(hx_ctx *ctx, const hx_model *model, const hx_calls *calls,
                     const hx_prefill_tab *pre, const hx_decode_tab *dec, const hx_links *links,
                     const float *tail, const float *horizon, int32_t n_nodes, int32_t n_wf,
                     int32_t *best_p, int32_t *best_d, float *best_cost, float *ratio,
                     const HxHorizonsPlan *reveal, bool *revealed, void *stream_)
{
    *revealed = false;
    return score_placements(ctx, model, calls, pre, dec, links, tail, horizon, n_nodes, n_wf, nullptr, nullptr,
                            best_p, best_d, best_cost, ratio, reveal, nullptr, revealed, stream_);
}

// The walks of an append that has begun and hx_score_placements (fused outputs) in one launch (*merged; otherwise
// nothing has been launched).  ratio: checked, not written, as above.
int hx_relax_search(hx_ctx *ctx, const hx_model *model, const hx_calls *calls,
                    const hx_prefill_tab *pre, const hx_decode_tab *dec, const hx_links *links,
                    const float *tail, const float *horizon, int32_t n_nodes, int32_t n_wf,
                    int32_t *best_p, int32_t *best_d, float *best_cost, float *ratio,
                    const HxAppendPlan *walks, bool *merged, void *stream_)
{
    *merged = false;
    return score_placements(ctx, model, calls, pre, dec, links, tail, horizon, n_nodes, n_wf, nullptr, nullptr,
                            best_p, best_d, best_cost, ratio, nullptr, walks, merged, stream_);
}

extern "C" int hx_select(hx_ctx *ctx, int32_t C, int32_t P, int32_t D, const float *cost,
                         const hx_calls *calls, const float *tail, const float *horizon,
                         int32_t n_nodes, int32_t n_wf,
                         int32_t *best_p, int32_t *best_d, float *best_cost, float *ratio, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HX_REQUIRE(ctx, C >= 0 && P >= 0 && D >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, (long long)P * D <= 2147483647LL, HX_ERR_SHAPE, "P*D beyond int32");
    HX_REQUIRE(ctx, best_p && best_d && best_cost, HX_ERR_INVALID_ARG, "NULL output");
    HX_REQUIRE(ctx, cost || (long long)C * P * D == 0, HX_ERR_INVALID_ARG, "cost is NULL");
    if (int rc = check_ratio_inputs(ctx, calls, tail, horizon, n_nodes, n_wf, ratio)) return rc;
    HX_REQUIRE(ctx, !calls || calls->n == C, HX_ERR_INVALID_ARG, "calls.n differs from C");
    if (C == 0) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;
    ScoreArgs a{};
    a.C = C; a.P = P; a.D = D; a.cost = const_cast<float *>(cost);
    if (calls) { a.node = calls->node; a.wf = calls->wf; a.elapsed = calls->elapsed; }
    a.tail = tail; a.horizon = horizon; a.n_nodes = n_nodes; a.n_wf = n_wf;
    a.best_p = best_p; a.best_d = best_d; a.best_cost = best_cost; a.ratio = ratio; a.status = ctx->d_status;
    const int most = ctx->num_cu * 8;
    const bool quads = ((long long)P * D & 3) == 0 && (reinterpret_cast<uintptr_t>(cost) & 15) == 0;
    if (quads && (long long)P * D <= SELECT_WAVE) {
        const int grid = C / 4 + (C % 4 != 0);
        if (P * D <= 4 * HX_WAVE) hx_select_wave_kernel<1><<<grid < most ? grid : most, 256, 0, stream>>>(a);
        else hx_select_wave_kernel<8><<<grid < most ? grid : most, 256, 0, stream>>>(a);
        return hx_check_launch(ctx, "hx_select_wave_kernel");
    }
    const int grid = C < most ? C : most;
    hx_select_kernel<<<grid, 256, 0, stream>>>(a);
    return hx_check_launch(ctx, "hx_select_kernel");
}

extern "C" int hx_urgency(hx_ctx *ctx, const hx_calls *calls, const float *best_cost,
                          const float *tail, const float *horizon, int32_t n_nodes, int32_t n_wf,
                          float *ratio, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HX_REQUIRE(ctx, calls, HX_ERR_INVALID_ARG, "NULL calls");
    const int C = calls->n;
    HX_REQUIRE(ctx, C >= 0 && n_nodes >= 0 && n_wf >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, C == 0 || (calls->node && calls->wf && calls->elapsed && best_cost && tail && horizon && ratio),
               HX_ERR_INVALID_ARG, "the ratio needs node, wf, elapsed, best_cost, tail and horizon");
    if (C == 0) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hx_urgency_kernel<<<(C + 255) / 256, 256, 0, (hipStream_t)stream_>>>(calls->node, calls->wf, calls->elapsed, best_cost, tail, horizon,
                                                                       n_nodes, n_wf, C, ratio, ctx->d_status);
    return hx_check_launch(ctx, "hx_urgency_kernel");
}
