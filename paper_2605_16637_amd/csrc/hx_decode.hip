// The decode stage (Sec. 5.4): calls whose KV has arrived wait for decode
// admission.  A call needs L_in + L_out tokens of KV (Eq. 3) under the
// instance's capacity (Eq. 4) for as long as it decodes; each instance carries
// token-capacity intervals (who holds how many tokens from when to when), and
// the earliest capacity-feasible start on an instance is the first moment from
// which the call fits for its whole decode time.  Projected finish = that start
// + decode time (Sec. 5.1: waiting for decode capacity plus decode execution);
// a call locked to an instance during prefill planning may only go there.
//
// Per instance the intervals are turned into a timeline: the distinct event
// times >= now in increasing order with the occupancy from each time to the
// next.  A start is feasible when a run of consecutive timeline segments that
// all leave room covers the decode time; a run can only begin where occupancy
// drops, i.e. now or at the end of an interval.
#include "hx_common.hpp"
#include "hx_terms.hpp"
#include "hx_search.hpp"

#include <climits>
#include <cmath>

namespace {

typedef unsigned long long u64;

// ---- timeline of one instance, built in LDS by a whole workgroup --------------------

// scratch for 2*cnt + 1 events (the extra one is "now")
struct TlScratch {
    u64 *key;        // (time bits, end-before-start flag, event id): unique, orders the events
    int *delta;      // +tok at a start, -tok at an end
    float *ts;       // sorted: time
    int *ds;         //         delta
};

// compact timeline: entry i covers [t_i, t_{i+1}) (the last one has no end) with occupancy occ_i
struct Tl {
    int2 *e;         // (time bits, occupancy)
};

__host__ __device__ inline size_t hx_align16(size_t x) { return (x + 15) & ~(size_t)15; }

// The scans read whole groups of entries, one group ahead: a timeline of up to ne entries is
// stored in ne rounded up to a multiple of eight, plus sixteen, the rest filled with (never, empty).
__host__ __device__ inline int hx_tl_len(int ne) { return ((ne + 7) & ~7) + 16; }

__device__ inline TlScratch hx_carve_scratch(unsigned char *p, int ne)
{
    TlScratch w;
    w.key = (u64 *)p;                 p += hx_align16((size_t)ne * 8);
    w.delta = (int *)p;               p += hx_align16((size_t)ne * 4);
    w.ts = (float *)p;                p += hx_align16((size_t)ne * 4);
    w.ds = (int *)p;
    return w;
}
__host__ __device__ inline size_t hx_scratch_bytes(int ne)
{
    return hx_align16((size_t)ne * 8) + 3 * hx_align16((size_t)ne * 4);
}

template <bool COHERENT, typename T> __device__ __forceinline__ T hx_ld(const T *p)
{
    // COHERENT: the value may have been written by another wave of this workgroup a moment ago
    if (COHERENT) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}

// Counting against all of n keys, one key per group of `parts` neighbouring lanes: 4 or 2 lanes per key where the
// workgroup has that many threads to spare (a power of two, so a group lies inside a quad of lanes).
__device__ __forceinline__ int hx_count_parts(int n, int nthreads) { return 4 * n <= nthreads ? 4 : (2 * n <= nthreads ? 2 : 1); }

// the sum over the lanes of a group (lane moves inside the quad; every lane of the group is active)
__device__ __forceinline__ int hx_parts_sum(int r, int parts)
{
    if (parts >= 2) r += __builtin_amdgcn_update_dpp(0, r, 0xB1, 0xf, 0xf, false);      // quad_perm [1,0,3,2]
    if (parts >= 4) r += __builtin_amdgcn_update_dpp(0, r, 0x4E, 0xf, 0xf, false);      // quad_perm [2,3,0,1]
    return r;
}

// All threads of the workgroup (WAVE: all lanes of one wavefront) call this.  cnt entries of one instance -> compact
// timeline in `out`, its length in *n_out (LDS).  Ends the call with a barrier.
template <bool COHERENT, bool WAVE = false>
__device__ void hx_build_timeline(int cnt, const float *st, const float *en, const int32_t *tk,
                                  TlScratch w, Tl out, int *n_out, int32_t *status)
{
    const int tid = WAVE ? threadIdx.x & (HX_WAVE - 1) : threadIdx.x, nthreads = WAVE ? HX_WAVE : blockDim.x;
    auto sync = [] {
        if constexpr (WAVE) hx_wave_sync();
        else __syncthreads();
    };
    const int n_ev = 2 * cnt + 1;
    for (int i = tid; i < n_ev; i += nthreads) {
        float time = 0.0f;
        int delta = 0;
        unsigned is_end = 1;                               // event 0 is "now"
        if (i > 0) {
            const int j = (i - 1) >> 1;
            is_end = (unsigned)(i - 1) & 1u;
            const float s = hx_ld<COHERENT>(st + j), e = hx_ld<COHERENT>(en + j);
            const int k = hx_ld<COHERENT>(tk + j);
            if (s < e && k > 0) {                          // anything else (NaN times included) holds nothing
                const float x = is_end ? e : s;
                time = x > 0.0f ? x : 0.0f;                // the past is folded onto now
                delta = is_end ? -k : k;
            }
        }
        // at equal times starts sort before ends, so the last event of a time is an end if there is one
        w.key[i] = ((u64)__float_as_uint(time) << 32) | ((u64)is_end << 31) | (unsigned)i;
        w.delta[i] = delta;
    }
    sync();
    // position of every event = number of smaller keys (keys are unique); with threads to spare, the 2 or 4
    // neighbouring lanes of an event count a part of the keys each
    const int parts = hx_count_parts(n_ev, nthreads);
    const int share = ((n_ev + parts - 1) / parts + 7) & ~7;
    for (int i = tid / parts; i < n_ev; i += nthreads / parts) {
        const u64 ki = w.key[i];
        const int j_lo = min((tid & (parts - 1)) * share, n_ev), j_hi = min(j_lo + share, n_ev);
        int r = 0;
        int j = j_lo;
        for (; j + 8 <= j_hi; j += 8) {                   // eight independent reads in flight
            u64 kk[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) kk[u] = w.key[j + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) r += kk[u] < ki;
        }
        for (; j < j_hi; ++j) r += w.key[j] < ki;
        r = hx_parts_sum(r, parts);
        if ((tid & (parts - 1)) == 0) {
            w.ts[r] = __uint_as_float((unsigned)(ki >> 32));
            w.ds[r] = w.delta[i];
        }
    }
    sync();
    // one wavefront: running occupancy, and one entry per distinct time (the last event of that time)
    if (tid < HX_WAVE) {
        const int per = (n_ev + HX_WAVE - 1) / HX_WAVE;
        const int lo = min(tid * per, n_ev), hi = min(lo + per, n_ev);
        long long sum = 0;
        int heads = 0;
        for (int i = lo; i < hi; ++i) {
            sum += w.ds[i];
            heads += (i == n_ev - 1) || (w.ts[i + 1] != w.ts[i]);
        }
        long long psum = sum;
        int ph = heads;
#pragma unroll
        for (int off = 1; off < HX_WAVE; off <<= 1) {
            const long long o = __shfl_up(psum, off);
            const int oh = __shfl_up(ph, off);
            if (tid >= off) { psum += o; ph += oh; }
        }
        long long run = psum - sum;
        int pos = ph - heads;
        for (int i = lo; i < hi; ++i) {
            run += w.ds[i];
            if ((i == n_ev - 1) || (w.ts[i + 1] != w.ts[i])) {
                if (run > (long long)INT_MAX) hx_raise(status, HX_ERR_OVERFLOW);
                const int occ = run > (long long)INT_MAX ? INT_MAX : (int)run;
                out.e[pos] = make_int2(__float_as_int(w.ts[i]), occ);
                ++pos;
            }
        }
        if (tid == HX_WAVE - 1) *n_out = pos;
    }
    sync();
    for (int i = *n_out + tid; i < hx_tl_len(n_ev); i += nthreads) out.e[i] = make_int2(0x7f800000, 0);
    sync();
}

// ---- earliest capacity-feasible start, one lane per (call, instance) ------------------

struct HxSlot {
    float S;     // start, +inf if none
    bool found;
};

// thr = tokens the call may find occupied (capacity - demand), < 0: never fits.  T = decode time.
// Lanes of a wavefront may scan different timelines (e 16-byte aligned, padded as hx_tl_len says).
//
// Straight-line arithmetic per entry, no flags: rs is the start of the run of entries with room
// that the scan is in, +inf while it is in none (a run begins at the first entry with room:
// min(+inf, t_i) = t_i; inside a run t_i > rs leaves rs alone); the run is long enough once the next
// entry's time reaches rs + T, which cannot happen outside a run (rs + T = +inf, and the entry
// whose successor is "never" always has room: everything has ended by then).  Run starts only
// grow along the timeline, so the earliest start is the minimum over all hits.  The loop ends when
// every lane has its answer or has passed the end of its timeline.
// begin: a multiple of eight, the lane's first entry (0, or a place no start can lie before).
__device__ __forceinline__ HxSlot hx_earliest_start(const int2 *e, int n, int thr, float T, bool active, int begin = 0)
{
    const bool open = active && thr >= 0;
    float rs = INFINITY, ans = INFINITY;
#define HX_TL_STEP(cur_, occ_, nxt_)                                              \
    {                                                                             \
        rs = (occ_) <= thr ? fminf(rs, __int_as_float(cur_)) : INFINITY;          \
        ans = fminf(ans, __int_as_float(nxt_) >= rs + T ? rs : INFINITY);         \
    }
    // eight entries per step, the next eight already on their way (lanes that are through read entry 0 on)
    const int4 *q = reinterpret_cast<const int4 *>(e) + (begin >> 1);
    int4 c0 = q[0], c1 = q[1], c2 = q[2], c3 = q[3];
    for (int i0 = 0;; i0 += 8) {
        const bool going = open && begin + i0 < n && !(ans < INFINITY);
        if (__builtin_amdgcn_ballot_w64(going) == 0) break;
        const int at = going ? (i0 >> 1) + 4 : 0;
        const int4 n0 = q[at], n1 = q[at + 1], n2 = q[at + 2], n3 = q[at + 3];
        const float keep = ans;
        HX_TL_STEP(c0.x, c0.y, c0.z)
        HX_TL_STEP(c0.z, c0.w, c1.x)
        HX_TL_STEP(c1.x, c1.y, c1.z)
        HX_TL_STEP(c1.z, c1.w, c2.x)
        HX_TL_STEP(c2.x, c2.y, c2.z)
        HX_TL_STEP(c2.z, c2.w, c3.x)
        HX_TL_STEP(c3.x, c3.y, c3.z)
        HX_TL_STEP(c3.z, c3.w, n0.x)
        ans = going ? ans : keep;
        c0 = n0; c1 = n1; c2 = n2; c3 = n3;
    }
#undef HX_TL_STEP
    const bool found = open && ans < INFINITY;
    return HxSlot{found ? ans : INFINITY, found};
}

// ---- one scoring pass over (queue x instances) -----------------------------------------

struct DecodeArgs {
    HxModelF m;
    int Q, D, stride;
    const int32_t *L_in, *L_out, *lock;
    const float *d_flops, *d_hbm;
    const int32_t *d_used, *d_cap, *d_batch;
    const int32_t *iv_count;
    const float *iv_start, *iv_end;
    const int32_t *iv_tok;
    float *start, *cost;
    // The free calls (valid, not locked) of the queue in queue order: the queue is cut into D slices of `per`
    // calls, slice d's free calls are free_c[d*per ..], n_free[d] of them.  Unused when there are no locks.
    int32_t *free_c, *n_free;
    int per;
    // Best candidate of every call within each group of gd consecutive instances: [group][Q] each.
    int gd, n_groups;
    float *part_cost, *part_start;
    int32_t *part_d;
    // Pairs that the occupancy kernel tries: `tries` calls an instance, the n-th of all of them call (n & try_mask) * try_step.
    int tries, try_mask, try_step;
    int32_t *status;
};

// what a lane knows of its call on an instance
struct HxDecodeCand {
    float T;
    int thr;
    bool legal;
};

__device__ __forceinline__ HxDecodeCand hx_decode_candidate(const HxModelF &m, int L, int O, int lk, int d, int D,
                                                            const HxDecF &x, int cap, int32_t *status)
{
    HxDecodeCand c;
    bool ok = L >= 0 && O >= 0 && lk >= -1 && lk < D;
    if (!ok) hx_raise(status, HX_ERR_INDEX);
    c.legal = ok && (lk < 0 || lk == d);
    const HxCallF cf = hx_call_terms(m, ok ? L : 0, ok ? O : 0);
    c.T = hx_decode_time(cf, x.c1, x.c2, x.kB);
    const long long room = (long long)cap - ((long long)L + (long long)O);
    c.thr = (!ok || room < 0) ? -1 : (room > (long long)INT_MAX ? INT_MAX : (int)room);
    return c;
}

// How the scoring kernel searches an instance's timeline, decided here per instance.
constexpr int HX_TAB = 4096;          // entries of the first-room table at most
constexpr int HX_TAB_MAX_N = 512;     // timeline entries at most for the table (their occupancies are ranked all against all)
constexpr int HX_TAB_FLAG = 1 << 16;  // added to the stretch count in an instance's record: the table was written

struct TlOut {
    int2 *e;         // [D][nt] timeline entries, padded
    int *n;          // [D] entries
    int *seg;        // [D][nt] heads of the stretches, then n
    int2 *head;      // [D][nt] per stretch: (time of its head, rank of the head's occupancy), padded with (-inf, 0)
    int *sorted;     // [D][nt] the n occupancies in increasing order
    float *G;        // [D][HX_TAB] first-room table
    int *meta;       // [D][8] what the scoring kernel reads first of an instance: n, m (+flag), capacity, decode terms c1, c2, kB
    // for the search of the best alone
    int *least;      // [D][nt] least occupancy of an entry and those before it
    int *step;       // [2][D][4] what that leaves free at eight entries, in increasing order, and the time of the entry after each (hx_step_word)
};

// Workgroup d: everything the scoring kernel needs of instance d -- its timeline, built in LDS; the timeline's
// stretches of non-increasing occupancy; where that is small enough, the first-room table; a record of the
// instance's sizes and decode terms -- and the free calls among the d-th slice of the queue, in order.
constexpr int TL_THREADS = 512;
__global__ __launch_bounds__(TL_THREADS) void hx_decode_timeline_kernel(DecodeArgs a, TlOut o, int nt)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_n, s_m;
    const int tid = threadIdx.x;
    const int d = blockIdx.x;
    const int ne = 2 * a.stride + 1;
    TlScratch w = hx_carve_scratch(smem, ne);
    Tl tl;
    tl.e = (int2 *)(smem + hx_scratch_bytes(ne));
    int cnt = a.iv_count[d];
    if (cnt < 0 || cnt > a.stride) {
        if (tid == 0) hx_raise(a.status, HX_ERR_INDEX);
        cnt = cnt < 0 ? 0 : a.stride;
    }
    // this workgroup's slice of the queue (see below): its first calls are asked for now and used after the build
    const int c_lo = d * a.per, c_hi = min(a.Q, (d + 1) * a.per);
    const bool pre_in = a.lock && c_lo + tid < c_hi;
    const int pre_L = pre_in ? a.L_in[c_lo + tid] : 0, pre_O = pre_in ? a.L_out[c_lo + tid] : 0;
    const int pre_lk = pre_in ? a.lock[c_lo + tid] : -1;
    const size_t at = (size_t)d * a.stride;
    hx_build_timeline<false>(cnt, a.iv_start + at, a.iv_end + at, a.iv_tok + at, w, tl, &s_n, a.status);
    const int n = s_n;
    // Everything below is worked out in LDS and registers first and written to memory at the very end: a
    // barrier waits for the stores before it, and there are several barriers to come.

    // This workgroup's slice of the queue: its free calls, in order.  A thread keeps the place of its call of
    // the first 512 (few slices are longer) and writes it with the rest.
    int my_place = -1, n_free = 0;
    if (a.lock) {
        __shared__ int s_wave_n[TL_THREADS / HX_WAVE];
        const int lane = tid & (HX_WAVE - 1), wave = tid >> 6;
        for (int base = c_lo; base < c_hi; base += blockDim.x) {
            const int c = base + tid;
            const bool in = c < c_hi;
            const bool first = base == c_lo;
            const int L = first ? pre_L : (in ? a.L_in[c] : 0), O = first ? pre_O : (in ? a.L_out[c] : 0);
            const int lk = first ? pre_lk : (in ? a.lock[c] : -1);
            const bool ok = L >= 0 && O >= 0 && lk >= -1 && lk < a.D;
            if (!ok) hx_raise(a.status, HX_ERR_INDEX);
            const bool is_free = in && ok && lk < 0;
            const u64 mf = __builtin_amdgcn_ballot_w64(is_free);
            if (lane == 0) s_wave_n[wave] = __popcll(mf);
            __syncthreads();
            int before = n_free;
            for (int w2 = 0; w2 < wave; ++w2) before += s_wave_n[w2];
            const int place = before + __popcll(mf & ((1ull << lane) - 1ull));
            if (is_free) {
                if (first) my_place = place;
                else a.free_c[d * a.per + place] = c;
            }
            for (int w2 = 0; w2 < TL_THREADS / HX_WAVE; ++w2) n_free += s_wave_n[w2];
            __syncthreads();
        }
    }

    // Occupancy rises only where a planned interval starts; between two such entries it never rises.  The
    // heads of these stretches (entry 0 and every entry above its predecessor), in order, and n as the last one.
    // The builder's scratch is free again: seg_l, rank and sorted live there.
    short *seg_l = (short *)w.ds;
    if (tid < HX_WAVE) {
        const int per_lane = (n + HX_WAVE - 1) / HX_WAVE;
        const int lo = min(tid * per_lane, n), hi = min(lo + per_lane, n);
        int heads = 0;
        for (int i = lo; i < hi; ++i) heads += i == 0 || tl.e[i].y > tl.e[i - 1].y;
        int incl = heads;
#pragma unroll
        for (int off = 1; off < HX_WAVE; off <<= 1) {
            const int up = __shfl_up(incl, off);
            if (tid >= off) incl += up;
        }
        int pos = incl - heads;
        for (int i = lo; i < hi; ++i)
            if (i == 0 || tl.e[i].y > tl.e[i - 1].y) seg_l[pos++] = (short)i;
        if (tid == HX_WAVE - 1) { seg_l[incl] = (short)n; s_m = incl; }
    }
    // (occupancy, entry) as one key, for the ranks below
    for (int i = tid; i < n; i += blockDim.x) w.key[i] = ((u64)(unsigned)tl.e[i].y << 16) | (unsigned)i;
    __syncthreads();
    const int m = s_m;
    // Few stretches over a timeline of moderate length: the table below fits and the scoring kernel uses it.
    const bool table = n <= HX_TAB_MAX_N && m * (n + 1) <= HX_TAB;
    // Whether an entry leaves room for a call depends only on how the call's threshold ranks among the n
    // occupancies: with r = the number of occupancies <= threshold, entry i has room exactly when
    // rank_i = #{j : occ_j <= occ_i} is <= r.  The keys below an entry's own give its place in increasing
    // order, the keys below (occupancy + 1, 0) its rank.
    int *rank = w.delta, *sorted = (int *)w.ts;
    if (table) {
        const int parts = hx_count_parts(n, TL_THREADS);
        const int share = ((n + parts - 1) / parts + 7) & ~7;
        for (int i = tid / parts; i < n; i += TL_THREADS / parts) {
            const u64 mine = w.key[i], above = ((mine >> 16) + 1) << 16;
            const int j_lo = min((tid & (parts - 1)) * share, n), j_hi = min(j_lo + share, n);
            int place = 0, le = 0;
            int j = j_lo;
            for (; j + 8 <= j_hi; j += 8) {                // eight independent reads in flight
                u64 other[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) other[u] = w.key[j + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) { place += other[u] < mine; le += other[u] < above; }
            }
            for (; j < j_hi; ++j) { const u64 other = w.key[j]; place += other < mine; le += other < above; }
            place = hx_parts_sum(place, parts); le = hx_parts_sum(le, parts);
            if ((tid & (parts - 1)) == 0) {
                rank[i] = le;
                sorted[place] = (int)(mine >> 16);
            }
        }
        __syncthreads();
    }

    // ---- the last barrier is behind: everything goes to memory
    for (int i = tid; i < hx_tl_len(2 * cnt + 1); i += blockDim.x) o.e[(size_t)d * nt + i] = tl.e[i];
    for (int k = tid; k <= m; k += blockDim.x) o.seg[(size_t)d * nt + k] = (int)seg_l[k];
    if (my_place >= 0) a.free_c[d * a.per + my_place] = c_lo + tid;
    if (tid == 0) {
        o.n[d] = n;
        if (a.lock) a.n_free[d] = n_free;
        // the instance's decode terms are the same for every call: worked out here, once
        const HxDecF x = hx_decode_terms(a.m, a.d_used[d], a.d_batch[d], 0, 1.0f / a.d_flops[d], 1.0f / a.d_hbm[d]);
        int *meta = o.meta + 8 * d;
        meta[0] = n; meta[1] = table ? (m | HX_TAB_FLAG) : m; meta[2] = a.d_cap[d];
        meta[3] = __float_as_int(x.c1); meta[4] = __float_as_int(x.c2); meta[5] = __float_as_int(x.kB); meta[6] = 0; meta[7] = 0;
    }
    if (!table) return;
    for (int i = tid; i < n; i += blockDim.x) o.sorted[(size_t)d * nt + i] = sorted[i];
    for (int k = tid; k < hx_tl_len(m); k += blockDim.x)
        o.head[(size_t)d * nt + k] = k < m ? make_int2(tl.e[seg_l[k]].x, rank[seg_l[k]]) : make_int2((int)0xff800000u, 0);
    // G[k][r]: the time of the first entry of stretch k that has room at threshold rank r, +inf if none has.
    // Ranks never rise inside a stretch, so that entry is found by bisection.
    const int width = n + 1;
    for (int idx = tid; idx < m * width; idx += blockDim.x) {
        const int k = idx / width, r = idx - k * width;
        const int last = seg_l[k + 1];
        int lo = seg_l[k], hi = last;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (rank[mid] <= r) hi = mid; else lo = mid + 1;
        }
        o.G[(size_t)d * HX_TAB + idx] = lo < last ? __int_as_float(tl.e[lo].x) : INFINITY;
    }
}

// The same scan as hx_earliest_start for a timeline every lane of the wavefront shares.  The
// timeline was written by an earlier kernel and nothing writes it now, so it is read through the
// constant address space: with wave-uniform addresses the entries arrive as scalars, cost no vector
// memory or LDS traffic, and feed the vector arithmetic as scalar operands.  Eight entries per
// step, the next eight already on their way.
typedef int HxTlGroup __attribute__((ext_vector_type(16)));      // eight (time, occupancy) entries
typedef __attribute__((address_space(4))) const HxTlGroup *hx_tl_group_cp;

__device__ __forceinline__ float hx_earliest_start_shared(const int2 *__restrict__ e, int n, int thr, float T, bool active)
{
    const bool open = active && thr >= 0;
    float rs = INFINITY, ans = INFINITY;
#define HX_TL_STEP(cur_, occ_, nxt_)                                              \
    {                                                                             \
        rs = (occ_) <= thr ? fminf(rs, __int_as_float(cur_)) : INFINITY;          \
        ans = fminf(ans, __int_as_float(nxt_) >= rs + T ? rs : INFINITY);         \
    }
    const hx_tl_group_cp g = (hx_tl_group_cp)(unsigned long long)e;
    HxTlGroup cur = g[0];
    for (int i0 = 0; i0 < n; i0 += 8) {
        if (__builtin_amdgcn_ballot_w64(open && !(ans < INFINITY)) == 0) break;
        const HxTlGroup nxt = g[(i0 >> 3) + 1];
        // a lane that already has its answer keeps it: later hits have later starts
        HX_TL_STEP(cur[0], cur[1], cur[2])
        HX_TL_STEP(cur[2], cur[3], cur[4])
        HX_TL_STEP(cur[4], cur[5], cur[6])
        HX_TL_STEP(cur[6], cur[7], cur[8])
        HX_TL_STEP(cur[8], cur[9], cur[10])
        HX_TL_STEP(cur[10], cur[11], cur[12])
        HX_TL_STEP(cur[12], cur[13], cur[14])
        HX_TL_STEP(cur[14], cur[15], nxt[0])
        cur = nxt;
    }
#undef HX_TL_STEP
    return open ? ans : INFINITY;
}

// The start from the first-room table (see the timeline kernel).  r: the rank of the call's threshold.
// Stretch by stretch: a run that reaches a head lasted until then, which is where its length is tested
// (the entry-by-entry scan tests it at every entry, but a run long enough at an entry inside a stretch
// is still the same run, and long enough, at the next head or at the end); the run survives the head if
// the head has room; otherwise the next run begins at the stretch's first entry with room, G[k][r].
// Inside a run that entry is the head itself, later than the run's start, so one minimum serves both
// cases.  The same comparisons on the same values as the scan: the same start bit for bit.
// head: per stretch (time, rank) in groups of eight, read as scalars; G, sorted: LDS.
// first: the first eight heads, which the caller asked for ahead of time.
__device__ __forceinline__ float hx_earliest_start_table(const int2 *__restrict__ head, HxTlGroup first, const float *G,
                                                         const int *sorted, int n, int m, int thr, float T, bool active)
{
    const bool open = active && thr >= 0;
    int r = 0;
    {
        int lo = 0, hi = n;                                // first position of sorted[] above thr = #{occ <= thr}
        while (__builtin_amdgcn_ballot_w64(lo < hi) != 0) {
            const int mid = (lo + hi) >> 1;
            const bool le = sorted[min(mid, n - 1)] <= thr;
            if (lo < hi) { if (le) lo = mid + 1; else hi = mid; }
        }
        r = open ? lo : 0;                                 // rank 0: no entry has room
    }
    const float *Gr = G + r;
    const int width = n + 1;
    float rs = INFINITY, ans = INFINITY;
    // Eight stretches per step: their heads arrive as scalars, their table entries are read together.  Past the
    // last stretch the heads are (-inf, rank 0) and the table row is the last one again: no hit, the run
    // kept, and a minimum with a value that is already in it.
#define HX_HEAD_STEP(u_)                                                          \
    {                                                                             \
        ans = fminf(ans, __int_as_float(cur[2 * (u_)]) >= rs + T ? rs : INFINITY); \
        rs = cur[2 * (u_) + 1] <= r ? rs : INFINITY;                              \
        rs = fminf(rs, gv[u_]);                                                   \
    }
    const hx_tl_group_cp g = (hx_tl_group_cp)(unsigned long long)head;
    HxTlGroup cur = first;
    for (int k0 = 0; k0 < m; k0 += 8) {
        if (__builtin_amdgcn_ballot_w64(open && !(ans < INFINITY)) == 0) break;
        const HxTlGroup nxt = g[(k0 >> 3) + 1];
        float gv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) gv[u] = Gr[min(k0 + u, m - 1) * width];
        HX_HEAD_STEP(0) HX_HEAD_STEP(1) HX_HEAD_STEP(2) HX_HEAD_STEP(3)
        HX_HEAD_STEP(4) HX_HEAD_STEP(5) HX_HEAD_STEP(6) HX_HEAD_STEP(7)
        cur = nxt;
    }
#undef HX_HEAD_STEP
    ans = fminf(ans, INFINITY >= rs + T ? rs : INFINITY);  // the last run reaches the end of the timeline
    return open ? ans : INFINITY;
}

// The same result by stretches instead of entries.  Inside a stretch occupancy never rises, so the
// entries with room are its tail, found by bisection; a run that has begun continues through every
// later stretch whose head still has room and ends at the first head that has not, which is where
// its length is tested (a run long enough at any earlier entry is long enough there).  All
// comparisons are the ones the entry-by-entry scan makes, on the same values, so the start is the
// same bit for bit; the work per (call, instance) is a few operations per stretch plus the
// bisections instead of seven per entry.  e: the timeline in LDS; seg[0..m]: heads and n.
__device__ __forceinline__ float hx_earliest_start_stretches(const int2 *e, const int *seg, int n, int m, int thr, float T, bool active)
{
    const bool open = active && thr >= 0;
    float rs = INFINITY, ans = INFINITY;
    for (int k = 0; k < m; ++k) {
        if (__builtin_amdgcn_ballot_w64(open && !(ans < INFINITY)) == 0) break;
        const int first = seg[k], last = seg[k + 1];
        const int2 head = e[first];
        const bool head_room = head.y <= thr;
        // a run that reaches a head lasted until then (rs = +inf outside a run: no hit)
        ans = fminf(ans, __int_as_float(head.x) >= rs + T ? rs : INFINITY);
        rs = head_room ? rs : INFINITY;
        // lanes outside a run take the first entry with room in this stretch, if there is one
        const bool need = open && !(rs < INFINITY);
        if (__builtin_amdgcn_ballot_w64(need) != 0) {
            int lo = first, hi = last;
            while (__builtin_amdgcn_ballot_w64(need && lo < hi) != 0) {
                const int mid = (lo + hi) >> 1;
                const bool room = e[min(mid, n - 1)].y <= thr;
                if (lo < hi) { if (room) hi = mid; else lo = mid + 1; }
            }
            if (need && lo < last) rs = __int_as_float(e[lo].x);
        }
    }
    ans = fminf(ans, INFINITY >= rs + T ? rs : INFINITY);  // the last run reaches the end of the timeline
    return open ? ans : INFINITY;
}

// What the scoring kernel knows of an instance: one 32-byte record, written by the timeline kernel and read
// as scalars.
typedef int HxMetaRec __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(4))) const HxMetaRec *hx_meta_cp;

struct HxInst {
    int n, m_flag, cap;
    float c1, c2, kB;              // the instance's part of the decode time of a call (hx_decode_terms)
    __device__ __forceinline__ int m() const { return m_flag & (HX_TAB_FLAG - 1); }
    // with the table: a few operations per stretch.  Else few long stretches: search them; many short ones
    // (most entries are starts): the plain scan, straight from memory.
    __device__ __forceinline__ bool by_table() const { return (m_flag & HX_TAB_FLAG) != 0; }
    __device__ __forceinline__ bool by_stretch() const { return !by_table() && 4 * m() <= n; }
};

__device__ __forceinline__ HxInst hx_inst_load(const TlOut &o, int d)
{
    const HxMetaRec r = ((hx_meta_cp)(unsigned long long)o.meta)[d];
    HxInst it;
    it.n = r[0]; it.m_flag = r[1]; it.cap = r[2];
    it.c1 = __int_as_float(r[3]); it.c2 = __int_as_float(r[4]); it.kB = __int_as_float(r[5]);
    return it;
}

// An instance's tables, copied to LDS by the whole workgroup.  With the table: its cells, then the sorted
// occupancies; for the stretch search: the timeline's (time, occupancy) pairs, then the stretch heads.
constexpr int DS_THREADS = 256;
constexpr int DS_OFF_SORTED = HX_TAB, DS_OFF_SEG = 2 * (2 * HX_MAX_INTERVALS + 2);   // words into the staging buffer
constexpr int DS_BUF = HX_TAB + HX_TAB_MAX_N;
static_assert(DS_BUF >= DS_OFF_SEG + HX_MAX_INTERVALS + 2, "the stretch search's arrays fit in the table's place");

// n words from memory to LDS by the whole workgroup, eight loads per thread asked for before the first is
// stored (one memory round trip per 2048 words); from[0] must be readable
__device__ __forceinline__ void hx_copy_words(int *to, const int *__restrict__ from, int n, int tid)
{
    for (int base = 0; base < n; base += 8 * DS_THREADS) {
        int v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * DS_THREADS + tid;
            v[u] = from[i < n ? i : 0];                    // past the end: the first word again, not stored
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * DS_THREADS + tid;
            if (i < n) to[i] = v[u];
        }
    }
}

__device__ __forceinline__ void hx_inst_stage(int *buf, const TlOut &o, int d, int nt, const HxInst &it, int tid)
{
    const int n = it.n, m = it.m();
    if (it.by_table()) {
        // the sorted occupancies (at most two per thread) ride with the table's first 2048 cells: one round trip
        const int *G = (const int *)(o.G + (size_t)d * HX_TAB), *sorted = o.sorted + (size_t)d * nt;
        const int cells = m * (n + 1);
        int v[8], s2[2];
#pragma unroll
        for (int u = 0; u < 8; ++u) { const int i = u * DS_THREADS + tid; v[u] = G[i < cells ? i : 0]; }
#pragma unroll
        for (int u = 0; u < 2; ++u) { const int i = u * DS_THREADS + tid; s2[u] = sorted[i < n ? i : 0]; }
#pragma unroll
        for (int u = 0; u < 8; ++u) { const int i = u * DS_THREADS + tid; if (i < cells) buf[i] = v[u]; }
#pragma unroll
        for (int u = 0; u < 2; ++u) { const int i = u * DS_THREADS + tid; if (i < n) buf[DS_OFF_SORTED + i] = s2[u]; }
        if (cells > 8 * DS_THREADS) hx_copy_words(buf + 8 * DS_THREADS, G + 8 * DS_THREADS, cells - 8 * DS_THREADS, tid);
    } else if (it.by_stretch()) {
        hx_copy_words(buf, (const int *)(o.e + (size_t)d * nt), 2 * n, tid);
        hx_copy_words(buf + DS_OFF_SEG, o.seg + (size_t)d * nt, m + 1, tid);
    }
}
static_assert(HX_TAB_MAX_N <= 2 * DS_THREADS, "two sorted occupancies per thread");

// Selection without atomics: a workgroup takes 256 free calls, one per lane, through a group of gd consecutive
// instances, one instance after the other, and every lane keeps the best (finish, instance, start) it has
// seen -- instances ascend, so "strictly smaller" keeps the lowest instance among equal finishes.  The lane's
// result for the group goes to part_*[group][call]; the finish kernel takes the minimum over the groups in
// the same order.  (Asking for an instance's tables while the one before it is searched, into a second
// buffer, was measured and gained nothing: with four workgroups to a compute unit the waits are already
// covered, and the extra address arithmetic costs what the overlap saves.)
//
// The first n_lock workgroups of the grid are for the locked calls instead, one lane per call of the queue
// (lanes of free calls idle): a locked call has its one instance, so each lane reads that instance's
// timeline for itself, and its result is the call's result (group 0's place).
__global__ __launch_bounds__(DS_THREADS) void hx_decode_score_kernel(DecodeArgs a, TlOut o, int nt, int n_lock)
{
    __shared__ __align__(16) int s_buf[DS_BUF];
    int *s_pref = s_buf;                                   // free calls before each slice of the queue: done with before the buffer is filled
    static_assert(DS_BUF >= HX_MAX_INSTANCES + 1, "the slice prefixes fit in the staging buffer");
    __shared__ int s_wave_n[DS_THREADS / HX_WAVE];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < n_lock) {
        const int c = (int)blockIdx.x * DS_THREADS + tid;
        const bool in = c < a.Q;
        const int L = in ? a.L_in[c] : 0, O = in ? a.L_out[c] : 0;
        const int lk = in ? a.lock[c] : -1;
        const bool ok = L >= 0 && O >= 0 && lk >= -1 && lk < a.D;              // an error is already raised
        const bool legal = in && ok && lk >= 0;
        const int d = legal ? lk : 0;
        const HxDecF x = hx_decode_terms(a.m, a.d_used[d], a.d_batch[d], 0, 1.0f / a.d_flops[d], 1.0f / a.d_hbm[d]);
        const HxDecodeCand k = hx_decode_candidate(a.m, legal ? L : 0, legal ? O : 0, -1, d, a.D, x, a.d_cap[d], a.status);
        const HxSlot s = hx_earliest_start(o.e + (size_t)d * nt, o.n[d], k.thr, k.T, legal);
        const float v = s.S + k.T;
        const bool placed = legal && s.found && v < INFINITY;
        if (in && !(ok && lk < 0)) {                       // locked or invalid: this lane speaks for the call
            a.part_cost[c] = placed ? v : INFINITY;
            a.part_start[c] = placed ? s.S : INFINITY;
            a.part_d[c] = placed ? d : -1;
            for (int j = 0; j < a.D; ++j) {
                const bool here = legal && j == d;
                if (a.start) a.start[(size_t)c * a.D + j] = here ? s.S : INFINITY;
                if (a.cost) a.cost[(size_t)c * a.D + j] = (here && s.found) ? v : INFINITY;
            }
        }
        return;
    }
    const int b = (int)blockIdx.x - n_lock;
    const int tile = b / a.n_groups, grp = b - tile * a.n_groups;
    const int lane = tid & (HX_WAVE - 1), wave = tid >> 6;
    const int d_lo = grp * a.gd, d_hi = min(a.D, (grp + 1) * a.gd);
    // which call this lane has: position tile*256 + tid of the free calls
    int c = tile * DS_THREADS + tid;
    bool in = c < a.Q;
    if (a.lock) {
        // free calls before each slice: an inclusive scan of the D slice counts, four per thread
        int v[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int idx = tid * 4 + j;
            v[j] = idx < a.D ? a.n_free[idx] : 0;
            sum += v[j];
        }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < HX_WAVE; off <<= 1) {
            const int up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        if (lane == HX_WAVE - 1) s_wave_n[wave] = incl;
        __syncthreads();
        int run = incl - sum;
        for (int w2 = 0; w2 < wave; ++w2) run += s_wave_n[w2];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int idx = tid * 4 + j;
            if (idx < a.D) s_pref[idx] = run;
            run += v[j];
            if (idx == a.D - 1) s_pref[a.D] = run;
        }
        __syncthreads();
        const int n_all = s_pref[a.D];
        const int p = tile * DS_THREADS + tid;
        if (tile * DS_THREADS >= n_all) return;            // the whole workgroup: the grid is sized for a queue without locks
        in = p < n_all;
        // the last slice that begins at or before position p
        int lo = 0, hi = a.D - 1;
        while (__builtin_amdgcn_ballot_w64(lo < hi) != 0) {
            const int mid = (lo + hi + 1) >> 1;
            const bool le = s_pref[mid] <= p;
            if (lo < hi) { if (le) lo = mid; else hi = mid - 1; }
        }
        c = in ? a.free_c[lo * a.per + (p - s_pref[lo])] : 0;
    } else if (tile * DS_THREADS >= a.Q) {
        return;
    }
    const bool has = in;                                   // a call of its own: writes a result, if only "none"
    int L = in ? a.L_in[c] : 0, O = in ? a.L_out[c] : 0;
    if (!a.lock && (L < 0 || O < 0)) { hx_raise(a.status, HX_ERR_INDEX); in = false; }
    if (!in) { L = 0; O = 0; }
    const HxCallF cf = hx_call_terms(a.m, L, O);
    const long long need = (long long)L + (long long)O;
    float best_v = INFINITY, best_S = INFINITY;
    int best_d = -1;
    HxInst cur = hx_inst_load(o, d_lo);
    for (int d = d_lo; d < d_hi; ++d) {
        const int *buf = s_buf;
        __syncthreads();                                   // the slice prefixes, or the last instance's tables, are done with
        hx_inst_stage(s_buf, o, d, nt, cur, tid);
        // (scalars, on their way while the tables land: the first heads of this instance, the next instance's record)
        const HxTlGroup heads = *(hx_tl_group_cp)(unsigned long long)(o.head + (size_t)d * nt);
        const HxInst nxt = hx_inst_load(o, min(d + 1, d_hi - 1));
        __syncthreads();
        const float T = hx_decode_time(cf, cur.c1, cur.c2, cur.kB);
        const long long room = (long long)cur.cap - need;
        const int thr = room < 0 ? -1 : (room > (long long)INT_MAX ? INT_MAX : (int)room);
        const int n = cur.n, m = cur.m();
        const float S = cur.by_table()     ? hx_earliest_start_table(o.head + (size_t)d * nt, heads, (const float *)buf, buf + DS_OFF_SORTED,
                                                                     n, m, thr, T, in)
                        : cur.by_stretch() ? hx_earliest_start_stretches((const int2 *)buf, buf + DS_OFF_SEG, n, m, thr, T, in)
                                           : hx_earliest_start_shared(o.e + (size_t)d * nt, n, thr, T, in);
        const float v = S + T;                             // +inf when there is no start
        if (in) {
            if (a.start) a.start[(size_t)c * a.D + d] = S;
            if (a.cost) a.cost[(size_t)c * a.D + d] = S < INFINITY ? v : INFINITY;
            if (S < INFINITY && v < best_v) { best_v = v; best_S = S; best_d = d; }
        }
        cur = nxt;
    }
    if (has) {
        const size_t at = (size_t)grp * a.Q + c;
        a.part_cost[at] = best_v; a.part_start[at] = best_S; a.part_d[at] = best_d;
    }
}

struct DecodeFinishArgs {
    int Q, D, n_groups;
    const int32_t *L_in, *L_out, *lock;
    const float *part_cost, *part_start;
    const int32_t *part_d;
    const int32_t *node, *wf;
    const float *elapsed, *tail, *horizon;
    int n_nodes, n_wf;
    int32_t *best_d;
    float *best_start, *best_cost, *ratio;
    int32_t *status;
};

// the best of the groups' candidates (one place only for a call that is not free); n_groups = 0: there are no instances
__global__ __launch_bounds__(64) void hx_decode_finish_kernel(DecodeFinishArgs a)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.Q) return;
    int d = -1;
    float S = INFINITY, v = INFINITY;
    const int lk = a.lock ? a.lock[c] : -1;
    const bool is_free = a.L_in[c] >= 0 && a.L_out[c] >= 0 && lk == -1;
    const int groups = is_free ? a.n_groups : min(a.n_groups, 1);
    // groups ascend in instance: "strictly smaller" keeps the lowest instance among equal finishes
    int g_best = -1;
    int g = 0;
    for (; g + 8 <= groups; g += 8) {
        float pv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) pv[u] = a.part_cost[(size_t)(g + u) * a.Q + c];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (pv[u] < v) { v = pv[u]; g_best = g + u; }
    }
    for (; g < groups; ++g) {
        const float pv = a.part_cost[(size_t)g * a.Q + c];
        if (pv < v) { v = pv; g_best = g; }
    }
    if (g_best >= 0) {
        S = a.part_start[(size_t)g_best * a.Q + c];
        d = a.part_d[(size_t)g_best * a.Q + c];
    }
    a.best_d[c] = d; a.best_start[c] = S; a.best_cost[c] = v;
    if (a.ratio)
        hx_projected_ratio(a.node, a.wf, a.elapsed, a.tail, a.horizon, a.n_nodes, a.n_wf, c, v, a.status, a.ratio);
}

// ---- the best instance of every call, where nobody asks for the pairs ---------------------
//
// A pair costs its start plus its decode time, and no start is before the instance's first moment with room for the call, nor that
// before now.  So the decode time alone bounds the cost from below, and an instance whose bound is beyond the best cost found so
// far need not be looked at.  A wavefront takes a call, its lanes the instances, and looks at one instance after the other in
// the order of their bounds; that instance's timeline is then read by all lanes, an entry each.  After DB_CLOSER instances
// every bound is made a closer one, from what eight steps say of the room there has been (hx_step_word); after DB_EXACT those that
// still matter the closest, the first moment with room itself (a bisection a lane, between two of the steps); after DB_ALL -- room that is
// too short again and again -- every lane searches the instances it has left for itself.
// Of 8192 free calls on 256 instances with 113 to 137 entries each one in 1.13 instances is looked at with the steps, 3.3 by the decode
// time alone; where every instance is full for ten seconds 56 and 90, and 3 with the bisection.
//
// Where room comes in pieces that are too short for most calls no bound helps.  Whether it does is tried beforehand: the occupancy kernel
// looks at each instance for a few calls of the queue, and where for more than DB_EVERY_PAIR in sixteen of these pairs the first room there
// is lasts too short a time all workgroups take their calls through all instances instead (hx_decode_every_pair).
//
// What bounds it: instruction issue, some 200 vector and 200 scalar instructions a call, and the chain of a call's memory round trips,
// 2.9 and 1.9 us for the first and the second call of a wavefront.  Whole passes (us; the pairs all formed through tables of first moments
// with room, as hx_decode_score_kernel does; so; and without the last two of the following): 16384 calls, half of them locked, on 256 instances with 120
// intervals 89, 22.5, 22.2; 500 on 1024 with 50 76, 20.8, 20.0; 16384 on 512 with 60 120, 41, 61; 3000 on 100 with 120 37, 19.7, 20.7; 1000 on 32 with
// 500 85, 55, 52.  Full for ten seconds: the first 89, 50.5, 50.9; 500 on 300 with 250 107, 131, 145; 16384 on 300 84, 66, 106; 4000 on 512 52, 59, 84; 16384 on 1024
// 214, 162, 180.  In pieces of 0.3 s: 2000 on 64 with 28 20, 12, 29; 16384 on 256 with 28 73, 75, 330; 4000 on 1024 with 28 90, 113, 455; 300 on 1024 with
// 120 181, 90, 319.  What these two are: the pairs tried beforehand and eight instances a lane for 257 to 512.
// (Of 4 and 8 s, for which some of the calls are too long, it is slower than all pairs by tables: 3000 on 100 26, 29, 31; 300 on 64 20, 24, 24.)

// Up to some moment no more than `room` tokens have been free, and `time_bits` is when that may change: as the upper halves of two
// floats, the first as its complement.  A call that needs more than the room has no start before that time; by halves, as far as the two
// differ there, no start before a time that is not later.  Such a call's word, without a time and with the lower half set, is below this one.
__device__ __forceinline__ unsigned hx_step_word(unsigned room, int time_bits)
{
    return ~(__float_as_uint((float)room) | 0xffffu) | ((unsigned)time_bits >> 16);
}

// The earliest start on one timeline, by a wavefront: an entry a lane, 64 at a time.  A run of entries with room begins where the one
// before it has none, and is a start if the run's end, the next entry without room, is far enough: the comparisons of
// hx_earliest_start, which tests a run at each of its entries, at the last of them, whose successor is the latest.
// e: nt entries may be read, n of them count; next: the lane's of the first 64.  Uniform in everything but the lane.
__device__ __forceinline__ float hx_earliest_start_wave(const int2 *__restrict__ e, int nt, int2 next, int n, int thr, float T, int lane)
{
    float rs = INFINITY;                                   // where the run that is open begins
    for (int i0 = 0; i0 < n; i0 += HX_WAVE) {
        const int2 x = next;
        next = e[min(i0 + HX_WAVE + lane, nt - 1)];
        const bool in = i0 + lane < n;
        const float t = in ? __int_as_float(x.x) : INFINITY;      // behind the last entry: never, which ends every run
        const u64 room = __builtin_amdgcn_ballot_w64(in && x.y <= thr);
        const bool open = rs < INFINITY;
        if (open && room != ~0ull) {
            if (hx_lane_value(t, __builtin_ctzll(~room)) >= rs + T) return rs;
            rs = INFINITY;
        }
        const u64 starts = room & ~(room << 1) & ~(open ? 1ull : 0ull);
        if (starts == 0) continue;
        const u64 ends = ~room >> lane;
        const int len = ends ? __builtin_ctzll(ends) : HX_WAVE;
        const float t_end = __shfl(t, lane + len);         // (a run up to the last lane: not looked at)
        const u64 hits = __builtin_amdgcn_ballot_w64(((starts >> lane) & 1) != 0 && lane + len < HX_WAVE && t_end >= t + T);
        if (hits) return hx_lane_value(t, __builtin_ctzll(hits));
        if (room >> (HX_WAVE - 1)) rs = hx_lane_value(t, HX_WAVE - 1 - __builtin_clzll(starts));
    }
    return rs;                                             // it lasts
}

// Whether the first run of entries with room is too short, so that there is room before the earliest start: that run alone is read.
__device__ __forceinline__ bool hx_first_room_short(const int2 *e, int n, int thr, float T, int lane)
{
    float from = INFINITY;
    for (int i0 = 0; i0 < n; i0 += HX_WAVE) {
        const int2 x = e[min(i0 + lane, n - 1)];
        const u64 room = __builtin_amdgcn_ballot_w64(i0 + lane < n && x.y <= thr);
        int first = 0;
        if (!(from < INFINITY)) {
            if (room == 0) continue;
            first = __builtin_ctzll(room);
            from = hx_lane_value(__int_as_float(x.x), first);
        }
        const u64 ends = ~room >> first;
        if (ends == 0) continue;
        const int end = first + __builtin_ctzll(ends);
        return i0 + end < n && hx_lane_value(__int_as_float(x.x), end) < from + T;
    }
    return false;
}

// What is said of a pair that has been tried: there is room for the call some time; the first there is lasts too short a time.
constexpr unsigned DB_FITS = 1, DB_SHORT = 2;
constexpr int DB_TRIES = 256;              // pairs tried, but at least one and at most seven an instance

// Workgroup d: the occupancy of instance d over time, an entry an event that lies ahead; those that lie behind (most sequences
// have begun) only add to what is held now.  Several events of one moment are several entries, all with what is held
// after the last.  No running sum: an event adds up those not after it while it counts those before it.
// Bound: two memory round trips (the record, the intervals) and the comparisons, n^2 of them on one compute unit.  50 registers: with more
// than 64 1024 workgroups are no longer resident together (500 calls on 1024 instances 16.3 -> 17.9 us).
constexpr int DO_THREADS = 512;
constexpr int DO_EVENTS = 2 * HX_MAX_INTERVALS + 42;      // and a filler for the shares of several lanes
static_assert(HX_MAX_INTERVALS <= DO_THREADS, "an interval a thread");
__global__ __launch_bounds__(DO_THREADS) void hx_decode_occupancy_kernel(DecodeArgs a, TlOut o, int nt)
{
    __shared__ __align__(16) u64 s_key[DO_EVENTS];         // time, event: unique
    __shared__ __align__(16) int s_delta[DO_EVENTS];
    __shared__ __align__(16) int2 s_e[2 * HX_MAX_INTERVALS + 1];
    __shared__ int s_least[2 * HX_MAX_INTERVALS + 1];
    __shared__ u64 s_now, s_all;                           // tokens held now; now or later
    __shared__ int s_n;
    __shared__ int2 s_try[DO_THREADS / HX_WAVE];           // of the call a wavefront tries: its time, and what may be held
    const int tid = threadIdx.x, lane = tid & (HX_WAVE - 1), d = blockIdx.x;
    // the intervals are asked for before it is known how many there are
    const size_t at = (size_t)d * a.stride + tid;
    const bool room = tid < a.stride;
    const float st = room ? a.iv_start[at] : 0.0f, en = room ? a.iv_end[at] : 0.0f;
    const int tk = room ? a.iv_tok[at] : 0;
    int cnt = a.iv_count[d];
    const float flops = a.d_flops[d], hbm = a.d_hbm[d];
    const int used = a.d_used[d], batch = a.d_batch[d], cap = a.d_cap[d];
    // the last `tries` wavefronts (never the first) try a call of the queue each: the last have the fewest intervals
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nth = DO_THREADS / HX_WAVE - 1 - wave;
    const bool tries = nth < a.tries;
    int L = 0, O = 0;
    if (tries) {
        int c = ((d * a.tries + nth) & a.try_mask) * a.try_step;
        asm("" : "+v"(c));                                 // vector loads: nobody waits for them with the scalar ones
        L = a.L_in[c]; O = a.L_out[c];
    }
    for (int i = tid; i < DO_EVENTS; i += DO_THREADS) { s_key[i] = ~0ull; s_delta[i] = 0; }
    if (tid == 0) { s_now = 0; s_all = 0; s_n = 0; }
    __syncthreads();
    if (cnt < 0 || cnt > a.stride) {
        if (tid == 0) hx_raise(a.status, HX_ERR_INDEX);
        cnt = cnt < 0 ? 0 : a.stride;
    }
    // anything else (NaN times included) holds nothing, and what has ended holds nothing any more
    const bool holds = tid < cnt && st < en && tk > 0 && en > 0.0f;
    const bool later = holds && st > 0.0f;
    const u64 m_end = __builtin_amdgcn_ballot_w64(holds), m_start = __builtin_amdgcn_ballot_w64(later);
    if (m_end) {
        const u64 sum_now = hx_wave_sum_i31(holds && !later ? tk : 0), sum_all = hx_wave_sum_i31(holds ? tk : 0);
        int first = 0;
        if (lane == 0) {
            first = atomicAdd(&s_n, __popcll(m_end) + __popcll(m_start));
            atomicAdd(&s_now, sum_now); atomicAdd(&s_all, sum_all);
        }
        first = __builtin_amdgcn_readfirstlane(first);
        const u64 below = (1ull << lane) - 1ull;
        const int i_end = first + __popcll(m_end & below), i_start = first + __popcll(m_end) + __popcll(m_start & below);
        if (holds) { s_key[i_end] = ((u64)__float_as_uint(en) << 32) | (unsigned)i_end; s_delta[i_end] = -tk; }
        if (later) { s_key[i_start] = ((u64)__float_as_uint(st) << 32) | (unsigned)i_start; s_delta[i_start] = tk; }
    }
    if (tries) {                                           // (while others gather the events)
        const HxDecF x = hx_decode_terms(a.m, used, batch, 0, 1.0f / flops, 1.0f / hbm);
        if (lane == 0) {
            const float T = hx_decode_time(hx_call_terms(a.m, L, O), x.c1, x.c2, x.kB);
            const bool fits = L >= 0 && O >= 0 && hx_fits(L, O, cap);
            s_try[nth] = make_int2(__float_as_int(T), fits ? (int)((long long)cap - ((long long)L + O)) : -1);
            if (nth == 0) {
                int *const meta = o.meta + 8 * d;
                *(int4 *)meta = make_int4(0, 0, cap, __float_as_int(x.c1));
                *(int2 *)(meta + 4) = make_int2(__float_as_int(x.c2), __float_as_int(x.kB));
            }
        }
    }
    __syncthreads();
    const int n = s_n;
    const u64 held = s_now;
    auto clamped = [&](long long occ) {
        if (occ > (long long)INT_MAX) { hx_raise(a.status, HX_ERR_OVERFLOW); occ = INT_MAX; }
        return (int)occ;
    };
    if (tid == 0) s_e[0] = make_int2(0, clamped((long long)held));
    if (s_all <= (u64)INT_MAX) {                           // every occupancy fits 32 bits
        const int parts = hx_count_parts(n, DO_THREADS);
        const int share = ((n + parts - 1) / parts + 7) & ~7;
        for (int i = tid / parts; i < n; i += DO_THREADS / parts) {
            const u64 mine = s_key[i];
            const int t = (int)(mine >> 32), after = t + 1;      // (no time's bits are negative)
            int place = 0, sum = 0;
            const int j_lo = (tid & (parts - 1)) * share;
            // (Past the last event the filler: before none, no tokens.  Whether an event is not after this one's moment is asked by
            // a difference's sign: a comparison is widened to 64 bits, at 66 registers, or waits for the one condition register.)
            for (int j = j_lo; j < j_lo + share; j += 8) {
                u64 key[8];
                int delta[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) { key[u] = s_key[j + u]; delta[u] = s_delta[j + u]; }
#pragma unroll
                for (int u = 0; u < 8; ++u) { place += key[u] < mine; sum += delta[u] & (((int)(key[u] >> 32) - after) >> 31); }
            }
            place = hx_parts_sum(place, parts); sum = hx_parts_sum(sum, parts);
            if ((tid & (parts - 1)) == 0) s_e[place + 1] = make_int2(t, (int)held + sum);
        }
    } else {
        for (int i = tid; i < n; i += DO_THREADS) {
            const u64 mine = s_key[i];
            const unsigned t = (unsigned)(mine >> 32);
            int place = 0;
            long long sum = 0;
            for (int j = 0; j < n; ++j) { place += s_key[j] < mine; sum += (unsigned)(s_key[j] >> 32) <= t ? s_delta[j] : 0; }
            s_e[place + 1] = make_int2((int)t, clamped((long long)held + sum));
        }
    }
    __syncthreads();
    const int n_e = n + 1;
    if (tid == DO_THREADS - HX_WAVE) o.meta[8 * d] = n_e;
    int2 *const e = o.e + (size_t)d * nt;
    for (int i = tid; i < hx_tl_len(n_e); i += DO_THREADS) e[i] = i < n_e ? s_e[i] : make_int2(0x7f800000, 0);
    if (tid < HX_WAVE) {
        const int per = (n_e + HX_WAVE - 1) / HX_WAVE, lo = min(tid * per, n_e), hi = min(lo + per, n_e);
        int least = INT_MAX;
        for (int i = lo; i < hi; ++i) least = min(least, s_e[i].y);
#pragma unroll
        for (int off = 1; off < HX_WAVE; off <<= 1) {
            const int up = __shfl_up(least, off);
            if (tid >= off) least = min(least, up);
        }
        int run = __shfl_up(least, 1);
        if (tid == 0) run = INT_MAX;
        for (int i = lo; i < hi; ++i) { run = min(run, s_e[i].y); s_least[i] = run; }
        hx_wave_sync();
        for (int i = tid; i < n_e; i += HX_WAVE) o.least[(size_t)d * nt + i] = s_least[i];
        if (tid < 8) {
            const int i = tid * n / 8;
            o.step[((tid >> 2) * a.D + d) * 4 + (tid & 3)] = n > 0 ? hx_step_word((unsigned)max((long long)cap - s_least[i], 0ll), s_e[i + 1].x) : 0;
        }
    }
    unsigned char *const says = (unsigned char *)(o.meta + 8 * d + 6) + wave;
    if (!tries) {
        if (lane == 0) *says = 0;
        return;
    }
    unsigned what = 0;
    const int thr = __builtin_amdgcn_readfirstlane(s_try[nth].y);      // tokens the call may find held, < 0: never fits
    if (thr >= 0) {
        const float T = hx_lane_value(__int_as_float(s_try[nth].x), 0);
        what = hx_first_room_short(s_e, n_e, thr, T, lane) ? DB_FITS | DB_SHORT : DB_FITS;
    }
    if (lane == 0) *says = (unsigned char)what;
}

constexpr int DB_THREADS = 256;
// Workgroups a compute unit at most: 4 16.0 us, 5 14.7, 6 13.8, 7 14.4, 8 14.8 (the last ones wait for a place).  Six also beyond 256 instances, where
// four and three have a place: with no more than these 16384 calls on 512 and 1024 full instances 76 -> 90 and 162 -> 187, others full for no time
// 26 -> 26 and 39 -> 36.5.
constexpr int DB_PER_CU = 6;
// (DB_EXACT 5, 6, 7: the first of the passes above 25.4, 22.6, 22.2, full for ten seconds 48.9, 50.5, 53.5; 500 on 1024 29.5, 20.8, 20.2; 16384 on 300 full ones
// 63, 66, 69.)
constexpr int DB_CLOSER = 1, DB_EXACT = 6, DB_ALL = 16;
// Every pair where more than so many sixteenths of those tried have room before their start: 3000 calls on 100 instances with 30 resident and 90
// planned intervals (some 8) 20 us, every pair 34; 300 on 33 with 64 and 191 (some 12) 22 and 37; in pieces of 4 s (12) 3000 on 100 29 and
// 16; of 2 s (14) 33 and 17.
constexpr unsigned DB_EVERY_PAIR = 13;

// The same where sixteen lanes, a row of the wavefront, search one timeline for sixteen calls: a lane loads an entry of sixteen and all
// of the row have it in turn.  e: nt entries may be read, n of them count.
__device__ __forceinline__ HxSlot hx_earliest_start_row(const int2 *__restrict__ e, int nt, int n, int thr, float T, bool active, int in_row)
{
    const bool open = active && thr >= 0;
    float rs = INFINITY, ans = INFINITY;
    int2 x = e[in_row];
    for (int i0 = 0;; i0 += 16) {
        const bool going = open && i0 < n && !(ans < INFINITY);
        if (__builtin_amdgcn_ballot_w64(going) == 0) break;
        const int2 next = e[i0 < n ? min(i0 + 16 + in_row, nt - 1) : 0];
        const float keep = ans;
#define HX_ROW(v_, u_) __builtin_amdgcn_update_dpp(0, v_, 0x150 + (u_), 0xf, 0xf, true)      // row_newbcast: all lanes take part
#define HX_TL_STEP(u_, nxt_)                                                                   \
        {                                                                                      \
            const int occ = HX_ROW(x.y, u_);                                                   \
            const float from = fminf(rs, __int_as_float(HX_ROW(x.x, u_))), then = __int_as_float(nxt_); \
            rs = occ <= thr ? from : INFINITY;                                                 \
            ans = fminf(ans, then >= rs + T ? rs : INFINITY);                                  \
        }
#define HX_TL_STEPS(u_) HX_TL_STEP(u_, HX_ROW(x.x, u_ + 1)) HX_TL_STEP(u_ + 1, HX_ROW(x.x, u_ + 2)) HX_TL_STEP(u_ + 2, HX_ROW(x.x, u_ + 3))
        HX_TL_STEPS(0) HX_TL_STEPS(3) HX_TL_STEPS(6) HX_TL_STEPS(9) HX_TL_STEPS(12)
        HX_TL_STEP(15, HX_ROW(next.x, 0))
#undef HX_TL_STEPS
#undef HX_TL_STEP
#undef HX_ROW
        ans = going ? ans : keep;                          // (past its own end a row goes over whatever lies there)
        x = next;
    }
    const bool found = open && ans < INFINITY;
    return HxSlot{found ? ans : INFINITY, found};
}

// All pairs of G (1, 4 or 16) calls from c0 on, by a workgroup: its lanes are G calls times instances.  Bound: the entries, nine instructions
// each, of sixteen calls; else, with few calls, the round trips of a lane's own timeline.
__device__ __forceinline__ void hx_decode_every_pair(const DecodeArgs &a, const DecodeFinishArgs &f, const TlOut &o, int nt, const int4 *s_inst,
                                                     float3 (*s_best)[16], int G, int c0)
{
    const int lane = threadIdx.x & (HX_WAVE - 1), wave = threadIdx.x / HX_WAVE;
    const int c = c0 + (lane & (G - 1));
    const bool in = c < a.Q;
    const int L = in ? a.L_in[c] : 0, O = in ? a.L_out[c] : 0, lk = in && a.lock ? a.lock[c] : -1;
    const bool ok = in && L >= 0 && O >= 0 && lk >= -1 && lk < a.D;
    const HxCallF cf = hx_call_terms(a.m, ok ? L : 0, ok ? O : 0);
    float best = INFINITY, best_S = INFINITY;
    int best_d = -1;
    for (int d = (int)threadIdx.x / G; __builtin_amdgcn_ballot_w64(d < a.D) != 0; d += DB_THREADS / G) {
        const int dl = min(d, a.D - 1);
        const int4 x = s_inst[dl];
        const int2 *e = o.e + (size_t)dl * nt;
        const int n = o.meta[8 * dl], thr = (int)((long long)x.w - ((long long)L + O));
        const float T = hx_decode_time(cf, __int_as_float(x.x), __int_as_float(x.y), __int_as_float(x.z));
        const bool on = ok && d < a.D && (lk < 0 || lk == d) && hx_fits(L, O, x.w) && T <= best;
        const HxSlot s = G == 16 ? hx_earliest_start_row(e, nt, n, thr, T, on, lane & 15) : hx_earliest_start(e, n, thr, T, on);
        const float v = s.S + T;
        if (on && v < best) { best = v; best_S = s.S; best_d = d; }
    }
    // the least; of equals the lowest instance
    auto take = [&](float v, float S, int d) {
        if (v < best || (v == best && (unsigned)d < (unsigned)best_d)) { best = v; best_S = S; best_d = d; }
    };
    for (int off = HX_WAVE / 2; off >= G; off >>= 1) {
        const float v = __shfl_xor(best, off), S = __shfl_xor(best_S, off);
        take(v, S, __shfl_xor(best_d, off));
    }
    if (lane < G) s_best[wave][lane] = make_float3(best, best_S, __int_as_float(best_d));
    __syncthreads();
    if ((int)threadIdx.x < G && in) {
        for (int w = 1; w < DB_THREADS / HX_WAVE; ++w) take(s_best[w][lane].x, s_best[w][lane].y, __float_as_int(s_best[w][lane].z));
        if (!ok) hx_raise(a.status, HX_ERR_INDEX);
        f.best_d[c] = best_d; f.best_start[c] = best_S; f.best_cost[c] = best;
        if (f.ratio) hx_projected_ratio(f.node, f.wf, f.elapsed, f.tail, f.horizon, f.n_nodes, f.n_wf, c, best, f.status, f.ratio);
    }
    __syncthreads();
}

// K: instances a lane
template <int K>
__global__ __launch_bounds__(DB_THREADS, K <= 4 ? 6 : K == 8 ? 4 : 3) void hx_decode_best_kernel(DecodeArgs a, DecodeFinishArgs f, TlOut o, int nt, int G)
{
    const int lane = threadIdx.x & (HX_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (DB_THREADS / HX_WAVE) + threadIdx.x / HX_WAVE));
    const int n_waves = gridDim.x * (DB_THREADS / HX_WAVE);
    // the lane's instances' decode terms and capacities: read from here where they are wanted, they cost no registers
    __shared__ __align__(16) int4 s_inst[K * HX_WAVE];
    unsigned tried = 0;                                    // of the pairs that the occupancy kernel has tried those that fit; in the upper half those with room too short
    for (int d = threadIdx.x; d < K * HX_WAVE; d += DB_THREADS) {
        const int4 *meta = (const int4 *)(o.meta + 8 * min(d, a.D - 1));
        const int4 x = meta[0], y = meta[1];
        s_inst[d] = make_int4(x.w, y.x, y.y, d < a.D ? x.z : -1);      // no instance: nothing fits
        if (d < a.D) tried += __popc(y.z & 0x01010101 * DB_FITS) + __popc(y.w & 0x01010101 * DB_FITS)
                              + ((__popc(y.z & 0x01010101 * DB_SHORT) + __popc(y.w & 0x01010101 * DB_SHORT)) << 16);
    }
    __shared__ unsigned s_tried[DB_THREADS / HX_WAVE];
    tried = hx_wave_sum(tried);
    if (lane == 0) s_tried[threadIdx.x / HX_WAVE] = tried;
    __shared__ __align__(16) uint4 s_step[2][K * HX_WAVE];
    for (int i = threadIdx.x; i < 2 * K * HX_WAVE; i += DB_THREADS)
        s_step[i / (K * HX_WAVE)][i % (K * HX_WAVE)] = ((const uint4 *)o.step)[i / (K * HX_WAVE) * a.D + min(i % (K * HX_WAVE), a.D - 1)];
    // What the next call says of itself travels while this one is placed: a lane each for L, O, lock, node, workflow and elapsed, and of the
    // results for instance, start, cost and ratio, so that either is one instruction.
    const int32_t *const none = a.L_in;                    // (of what there is not; not used)
    const int32_t *in = lane == 0 ? a.L_in : lane == 1 ? a.L_out : none;
    if (lane == 2 && a.lock) in = a.lock;
    if (f.ratio) in = lane == 3 ? f.node : lane == 4 ? f.wf : lane == 5 ? (const int32_t *)f.elapsed : in;
    int32_t *const out = lane == 0 ? f.best_d : lane == 1 ? (int32_t *)f.best_start : lane == 2 ? (int32_t *)f.best_cost : (int32_t *)f.ratio;
    const bool writes = lane < (f.ratio ? 4 : 3);
    int next = wave < a.Q ? in[wave] : 0;
    __syncthreads();
    tried = 0;
#pragma unroll
    for (int w = 0; w < DB_THREADS / HX_WAVE; ++w) tried += s_tried[w];
    if (__builtin_expect((tried >> 16) * 16u > (tried & 0xffffu) * DB_EVERY_PAIR, 0)) {
        __shared__ float3 s_best[DB_THREADS / HX_WAVE][16];
        for (int c0 = (int)blockIdx.x * G; c0 < a.Q; c0 += (int)gridDim.x * G) hx_decode_every_pair(a, f, o, nt, s_inst, s_best, G, c0);
        return;
    }
    for (int c = wave; c < a.Q; c += n_waves) {
        const int L = __builtin_amdgcn_readlane(next, 0), O = __builtin_amdgcn_readlane(next, 1);
        const int lk = a.lock ? __builtin_amdgcn_readlane(next, 2) : -1;
        const int nd = __builtin_amdgcn_readlane(next, 3), w = __builtin_amdgcn_readlane(next, 4);
        const float el = hx_lane_value(__int_as_float(next), 5);
        const bool ratio_ok = f.ratio && nd >= 0 && nd < f.n_nodes && w >= 0 && w < f.n_wf;
        float graph = 1.0f;                                // lane 0: the tail of its node, lane 1: the horizon of its workflow
        if (ratio_ok) graph = *(lane == 0 ? f.tail + nd : f.horizon + w);
        if (c + n_waves < a.Q) next = in[c + n_waves];
        const bool ok = L >= 0 && O >= 0 && lk >= -1 && lk < a.D;
        const HxCallF cf = hx_call_terms(a.m, ok ? L : 0, ok ? O : 0);
        const long long need = (long long)L + (long long)O;
        float best = INFINITY, best_S = INFINITY;
        int best_d = -1;
        auto threshold = [&](int cap_d) {                  // tokens the call may find held, < 0: never fits
            const long long left = (long long)cap_d - need;
            return left < 0 ? -1 : (left > (long long)INT_MAX ? INT_MAX : (int)left);
        };
        auto time_on = [&](const int4 &x) { return hx_decode_time(cf, __int_as_float(x.x), __int_as_float(x.y), __int_as_float(x.z)); };
        auto look = [&](int d) {
            const int2 *e = o.e + (size_t)d * nt;
            const int2 first = e[min(lane, nt - 1)];       // asked for beside the record
            const HxInst it = hx_inst_load(o, d);
            const float T = hx_decode_time(cf, it.c1, it.c2, it.kB);
            const int thr = threshold(it.cap);
            const float S = hx_earliest_start_wave(e, nt, first, it.n, thr, T, lane);
            const float v = S + T;                         // +inf when there is no start
            if (v < best || (v == best && d < best_d)) { best = v; best_S = S; best_d = d; }
        };
        if (ok && lk >= 0) look(lk);
        else if (ok) {
            float bound[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int4 x = s_inst[k * HX_WAVE + lane];
                bound[k] = hx_fits(L, O, x.w) ? time_on(x) : INFINITY;
            }
            for (int looked = 1;; ++looked) {
                float low = bound[0];
#pragma unroll
                for (int k = 1; k < K; ++k) low = fminf(low, bound[k]);
                low = hx_wave_min(low);
                if (!(low <= best) || !(low < INFINITY)) break;
                int d = INT_MAX;
#pragma unroll
                for (int k = K - 1; k >= 0; --k) {
                    const u64 b = __builtin_amdgcn_ballot_w64(bound[k] == low);
                    d = b ? k * HX_WAVE + __builtin_ctzll(b) : d;
                }
                if (low == best && d > best_d) break;      // it could only be as good, and is not the lower instance
                look(d);
#pragma unroll
                for (int k = 0; k < K; ++k) bound[k] = k * HX_WAVE + lane == d ? INFINITY : bound[k];
                if (looked == DB_ALL) {
                    float v = INFINITY, S = INFINITY;
                    int at = INT_MAX;
#pragma unroll 1
                    for (int d0 = 0; d0 < a.D; d0 += HX_WAVE) {
                        float b = INFINITY;
#pragma unroll
                        for (int k = 0; k < K; ++k) b = k * HX_WAVE == d0 ? bound[k] : b;
                        const bool on = b <= best && b < INFINITY;
                        // (the comparisons of hx_earliest_start)
                        const int dl = min(d0 + lane, a.D - 1);
                        const int4 x = s_inst[d0 + lane];
                        const int thr = threshold(x.w), n = on ? o.meta[8 * dl] : 0;
                        const float T = time_on(x);
                        const int4 *e = (const int4 *)(o.e + (size_t)dl * nt);
                        // (eight entries at a time: a lane's are the lines of its own instance, and a round trip brings them all)
                        float rs = INFINITY, got = INFINITY;
                        for (int i = 0; __builtin_amdgcn_ballot_w64(i < n && !(got < INFINITY)) != 0; i += 8) {
                            const int4 *g = e + (i < n ? i >> 1 : 0);
                            int4 q[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) q[u] = g[u];
                            const float after = __int_as_float(g[4].x), before = got;
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const float then = u < 3 ? __int_as_float(q[u < 3 ? u + 1 : 3].x) : after;
                                rs = q[u].y <= thr ? fminf(rs, __int_as_float(q[u].x)) : INFINITY;
                                got = fminf(got, __int_as_float(q[u].z) >= rs + T ? rs : INFINITY);
                                rs = q[u].w <= thr ? fminf(rs, __int_as_float(q[u].z)) : INFINITY;
                                got = fminf(got, then >= rs + T ? rs : INFINITY);
                            }
                            got = i < n ? got : before;
                        }
                        if (on && got + T < v) { v = got + T; S = got; at = dl; }
                    }
                    const float all = hx_wave_min(v);
                    const int d_all = hx_wave_min(v == all && all < INFINITY ? at : INT_MAX);
                    if (d_all != INT_MAX && (all < best || (all == best && d_all < best_d))) {
                        best = all; best_d = d_all;
                        best_S = hx_lane_value(S, d_all & (HX_WAVE - 1));
                    }
                    break;
                }
                if (looked == DB_CLOSER) {
                    // a closer bound: while the least that has been held leaves no room there is no start
                    const unsigned me = hx_step_word((unsigned)L + (unsigned)O, 0) | 0xffffu;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const uint4 x = s_step[0][k * HX_WAVE + lane], y = s_step[1][k * HX_WAVE + lane];
                        unsigned t = me < x.x ? x.x : 0u;
                        t = me < x.y ? x.y : t; t = me < x.z ? x.z : t; t = me < x.w ? x.w : t;
                        t = me < y.x ? y.x : t; t = me < y.y ? y.y : t; t = me < y.z ? y.z : t; t = me < y.w ? y.w : t;
                        bound[k] = __uint_as_float(t << 16) + bound[k];
                    }
                } else if (looked == DB_EXACT) {
                    // the closest, where the other one is not beyond the best: the instance's first entry with room
                    unsigned span[K];                      // the lowest place it may have, and above that the highest
                    bool any = false;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const bool on = bound[k] <= best && bound[k] < INFINITY;
                        const unsigned n = on ? o.meta[8 * (k * HX_WAVE + lane)] - 1 : 0;      // (the last entry has room: everything has ended)
                        // between the last step that surely leaves no room and the first that surely does
                        const unsigned me = ~__float_as_uint((float)((unsigned)L + (unsigned)O)) >> 16;
                        unsigned none = 0, perhaps = 0;
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const uint4 x = s_step[h][k * HX_WAVE + lane];
                            none += (x.x >> 16 > me) + (x.y >> 16 > me) + (x.z >> 16 > me) + (x.w >> 16 > me);
                            perhaps += (x.x >> 16 >= me) + (x.y >> 16 >= me) + (x.z >> 16 >= me) + (x.w >> 16 >= me);
                        }
                        span[k] = on ? (perhaps * n >> 3) << 16 | (none ? ((none - 1) * n >> 3) + 1 : 0) : 0;
                        any = any || on;
                    }
                    if (__builtin_amdgcn_ballot_w64(any) == 0) break;
                    for (;;) {
                        bool going = false;
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            const unsigned lo = span[k] & 0xffffu, hi = span[k] >> 16;
                            if (lo >= hi) continue;
                            const unsigned mid = (lo + hi) >> 1;
                            const bool room = o.least[(unsigned)(k * HX_WAVE + lane) * (unsigned)nt + mid] <= threshold(s_inst[k * HX_WAVE + lane].w);
                            span[k] = room ? mid << 16 | lo : hi << 16 | (mid + 1);
                            going = going || (room ? lo < mid : mid + 1 < hi);
                        }
                        if (__builtin_amdgcn_ballot_w64(going) == 0) break;
                    }
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const unsigned lo = span[k] & 0xffffu;
                        if (lo > 0) bound[k] = __int_as_float(o.e[(unsigned)(k * HX_WAVE + lane) * (unsigned)nt + lo].x) + time_on(s_inst[k * HX_WAVE + lane]);
                    }
                }
            }
        }
        if (!ok || (f.ratio && !ratio_ok)) {
            if (lane == 0) hx_raise(a.status, HX_ERR_INDEX);
        }
        const int ratio = (int)hx_ratio_bits(el, best, hx_lane_value(graph, 0), hx_lane_value(graph, 1), ratio_ok);
        const int result = lane == 0 ? best_d : lane == 1 ? __float_as_int(best_S) : lane == 2 ? __float_as_int(best) : ratio;
        if (writes) out[c] = result;
    }
}

// ---- recomputing greedy of the decode stage, one workgroup -----------------------------

constexpr int DG_THREADS = 1024;
constexpr int DG_WAVES = DG_THREADS / HX_WAVE;
constexpr int DP_MAX_THREADS = HX_DECODE_GREEDY_MAX_CALLS;   // a lane per call at least
constexpr int DP_THREADS = 512;
constexpr int DP_MAX_G = 4;                                  // lanes per call at most
constexpr int DP_TOGETHER = 60;                              // comparisons a lane that a timeline built by all wavefronts has to save
constexpr int DP_FEW = 12;                                   // calls of a wavefront whose starts are found one after the other (24: 705 us)

struct DGreedyArgs {
    HxModelF m;
    int Q, D, stride;
    const int32_t *L_in, *L_out, *lock, *node, *wf;
    const float *elapsed, *tail, *horizon;
    int n_nodes, n_wf;
    const float *d_flops, *d_hbm;
    const int32_t *d_used, *d_cap, *d_batch;
    int32_t *iv_count;
    float *iv_start, *iv_end;
    int32_t *iv_tok;
    int32_t *best_d, *rank;
    float *best_start, *best_cost, *ratio;
    int32_t *status;
};

// LDS carve-up shared by host (size) and device (offsets)
struct DGreedyLds {
    int ne, nt, D, Q;      // events per instance, stored timeline length, padded sizes
    __host__ __device__ DGreedyLds(int stride, int D_, int Q_)
        : ne(2 * stride + 1), nt(hx_tl_len(2 * stride + 1) + 2), D((D_ + 3) & ~3), Q((Q_ + 3) & ~3) {}
    // + 2: the lanes of a wavefront scan different timelines with 16-byte reads; with a timeline length of
    // 4k + 2 entries neighbouring timelines start 16 bytes apart modulo the banks instead of on the same ones
    __host__ __device__ size_t off_tl() const { return hx_scratch_bytes(ne); }
    __host__ __device__ size_t off_inst() const { return off_tl() + hx_align16((size_t)D * nt * 8); }
    __host__ __device__ size_t off_call() const { return off_inst() + (size_t)6 * D * 4; }
    __host__ __device__ size_t off_red() const { return off_call() + (size_t)11 * Q * 4; }
    __host__ __device__ size_t bytes() const { return hx_align16(off_red() + (size_t)(2 * DG_WAVES + 8) * 4); }
};

enum : int { DG_ALIVE = 1, DG_DIRTY = 2 };

// The plan where LDS has no room for the start of every (instance, call) pair.  An added interval can only delay starts on
// the instance that received it; everything else stands: a call is scored again, on every instance, if its instance
// is the one that changed.  The same plan as the kernel below makes: the same functions on the same timelines, the
// same (finish, instance) rule.
__global__ __launch_bounds__(DG_THREADS) void hx_decode_plan_lean_kernel(DGreedyArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const DGreedyLds lay(a.stride, a.D, a.Q);
    TlScratch w = hx_carve_scratch(smem, lay.ne);
    int2 *s_tl = (int2 *)(smem + lay.off_tl());
    int *s_n = (int *)(smem + lay.off_inst());
    int *s_cnt = s_n + lay.D;
    int *s_cap = s_cnt + lay.D;
    float *s_c1 = (float *)(s_cap + lay.D);
    float *s_c2 = s_c1 + lay.D;
    float *s_kB = s_c2 + lay.D;
    int *s_bd = (int *)(smem + lay.off_call());
    float *s_bs = (float *)(s_bd + lay.Q);
    float *s_bc = s_bs + lay.Q;
    unsigned *s_ratio = (unsigned *)(s_bc + lay.Q);       // bits: it may be the NaN
    int *s_flags = (int *)(s_ratio + lay.Q);
    int *s_L = s_flags + lay.Q;                            // what the queue says of a call, read once
    int *s_O = s_L + lay.Q;
    int *s_lk = s_O + lay.Q;
    float *s_el = (float *)(s_lk + lay.Q);
    float *s_tail = s_el + lay.Q;                          // tail of its node, horizon of its workflow (-1: index out of range)
    float *s_hz = s_tail + lay.Q;
    float *s_redv = (float *)(smem + lay.off_red());
    int *s_redi = (int *)(s_redv + DG_WAVES);
    int *s_pick = s_redi + DG_WAVES;

    const int tid = threadIdx.x;
    const int lane = tid & (HX_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    for (int d = tid; d < a.D; d += DG_THREADS) {
        int cnt = a.iv_count[d];
        if (cnt < 0 || cnt > a.stride) { hx_raise(a.status, HX_ERR_INDEX); cnt = cnt < 0 ? 0 : a.stride; }
        s_cnt[d] = cnt;
        s_cap[d] = a.d_cap[d];
        const HxDecF x = hx_decode_terms(a.m, a.d_used[d], a.d_batch[d], 0, 1.0f / a.d_flops[d], 1.0f / a.d_hbm[d]);
        s_c1[d] = x.c1; s_c2[d] = x.c2; s_kB[d] = x.kB;
    }
    for (int c = tid; c < a.Q; c += DG_THREADS) {
        s_flags[c] = DG_ALIVE | DG_DIRTY;
        s_L[c] = a.L_in[c]; s_O[c] = a.L_out[c]; s_lk[c] = a.lock ? a.lock[c] : -1; s_el[c] = a.elapsed[c];
        const int nd = a.node[c], w = a.wf[c];
        const bool ok = nd >= 0 && nd < a.n_nodes && w >= 0 && w < a.n_wf;
        if (!ok) hx_raise(a.status, HX_ERR_INDEX);
        s_tail[c] = ok ? a.tail[nd] : 0.0f;
        s_hz[c] = ok ? fmaxf(a.horizon[w], 0.0f) : -1.0f;
    }
    __syncthreads();
    for (int d = 0; d < a.D; ++d) {
        const size_t at = (size_t)d * a.stride;
        Tl tl{s_tl + (size_t)d * lay.nt};
        hx_build_timeline<false>(s_cnt[d], a.iv_start + at, a.iv_end + at, a.iv_tok + at, w, tl, &s_n[d], a.status);
    }

    for (int k = 0; k < a.Q; ++k) {
        // (1) score the calls whose instance changed: one wavefront per call, lanes over instances
        for (int c = wave; c < a.Q; c += DG_WAVES) {
            if (s_flags[c] != (DG_ALIVE | DG_DIRTY)) continue;     // wave-uniform
            const int L = s_L[c], O = s_O[c];
            const int lk = s_lk[c];
            float bv = INFINITY, bS = INFINITY;
            int bd = INT_MAX;
            for (int d0 = 0; d0 < a.D; d0 += HX_WAVE) {
                const int d = d0 + lane;
                const bool in = d < a.D;
                const int dd = in ? d : 0;
                HxDecF x;
                x.wait = 0.0f; x.c1 = s_c1[dd]; x.c2 = s_c2[dd]; x.kB = s_kB[dd];
                const HxDecodeCand q = hx_decode_candidate(a.m, L, O, lk, dd, a.D, x, s_cap[dd], a.status);
                const HxSlot s = hx_earliest_start(s_tl + (size_t)dd * lay.nt, s_n[dd],
                                                   q.thr, q.T, in && q.legal);
                const float v = s.S + q.T;
                if (in && s.found && v < bv) { bv = v; bS = s.S; bd = d; }
            }
            const float best = hx_wave_min(bv);
            const int best_d = hx_wave_min(bv == best && best < INFINITY ? bd : INT_MAX);
            const float best_S = __shfl(bS, best_d == INT_MAX ? 0 : (best_d & (HX_WAVE - 1)));
            if (lane == 0) {
                const bool any = best_d != INT_MAX;
                s_bd[c] = any ? best_d : -1;
                s_bs[c] = any ? best_S : INFINITY;
                s_bc[c] = any ? best : INFINITY;
                s_ratio[c] = hx_ratio_bits(s_el[c], any ? best : INFINITY, s_tail[c], s_hz[c], s_hz[c] >= 0.0f);   // Eq. (2)
                s_flags[c] = DG_ALIVE;
            }
        }
        __syncthreads();
        // (2) the most urgent remaining call: largest ratio, lowest index among equals
        float rv = -INFINITY;
        int ri = INT_MAX;
        for (int c = tid; c < a.Q; c += DG_THREADS) {
            if (s_flags[c] & DG_ALIVE) {
                const float r = hx_rank_key(s_ratio[c]);
                if (ri == INT_MAX || r > rv) { rv = r; ri = c; }
            }
        }
        hx_wave_argmax(rv, ri);
        if (lane == 0) { s_redv[wave] = rv; s_redi[wave] = ri; }
        __syncthreads();
        // (3) the first wavefront takes the best of the wavefronts' candidates (one per lane, the same rule), and its
        // first lane records the pick and appends its interval
        if (wave == 0) {
            rv = lane < DG_WAVES ? s_redv[lane] : -INFINITY;
            ri = lane < DG_WAVES ? s_redi[lane] : INT_MAX;
            hx_wave_argmax(rv, ri);
        }
        if (tid == 0) {
            const int c = ri, d = s_bd[c];
            a.best_d[c] = d; a.best_start[c] = s_bs[c]; a.best_cost[c] = s_bc[c]; hx_store_bits(a.ratio, c, s_ratio[c]); a.rank[c] = k;
            s_flags[c] = 0;
            int changed = -1;
            if (d >= 0) {
                if (s_cnt[d] >= a.stride) {
                    hx_raise(a.status, HX_ERR_CAPACITY);
                } else {
                    const size_t at = (size_t)d * a.stride + s_cnt[d];
                    const long long need = (long long)s_L[c] + (long long)s_O[c];
                    a.iv_start[at] = s_bs[c];
                    a.iv_end[at] = s_bc[c];
                    a.iv_tok[at] = need > (long long)INT_MAX ? INT_MAX : (int)need;
                    s_cnt[d] += 1;
                    changed = d;
                    // The usual case -- the interval holds something, starts now or later, ends at a finite time, and
                    // the timeline has at most one entry per thread -- is inserted into the timeline below;
                    // anything else has the timeline built again from the instance's intervals.
                    const float S = s_bs[c], E = s_bc[c];
                    s_pick[1] = (S >= 0.0f && S < E && E < INFINITY && need > 0 && s_n[d] <= DG_THREADS) ? 1 : 0;
                    if (!s_pick[1]) __threadfence();                 // the other threads are about to read the interval from memory
                    s_pick[2] = s_n[d]; s_pick[3] = s_n[d];          // entries before S, before E: all, unless an entry says otherwise
                    s_pick[4] = __float_as_int(S > 0.0f ? S : 0.0f); s_pick[5] = __float_as_int(E);
                    s_pick[6] = need > (long long)INT_MAX ? INT_MAX : (int)need;
                }
            }
            s_pick[0] = changed;
        }
        __syncthreads();
        // (4) the timeline of the instance that took the call, and who has to look again
        const int pd = s_pick[0];
        if (pd >= 0) {
            const size_t at = (size_t)pd * a.stride;
            Tl tl{s_tl + (size_t)pd * lay.nt};
            if (s_pick[1]) {
                // The compact timeline is a function of the instance's events, so adding the two events of the new
                // interval (S, E, tok) to it gives what building it again would: entries from S up to E hold tok
                // more; S and E become entries of their own unless the timeline already has an entry at that time
                // (S: the occupancy before it plus tok; E: the occupancy that stood before E).
                const int n = s_n[pd];
                const float S = __int_as_float(s_pick[4]), E = __int_as_float(s_pick[5]);
                const int tok = s_pick[6];
                const bool in = tid < n;
                const int2 me = in ? tl.e[tid] : make_int2(0x7f800000, 0);
                const float t = __int_as_float(me.x);
                const float before = (in && tid > 0) ? __int_as_float(tl.e[tid - 1].x) : -1.0f;
                if (in && t >= S && before < S) s_pick[2] = tid;
                if (in && t >= E && before < E) s_pick[3] = tid;
                __syncthreads();
                const int pos_s = s_pick[2], pos_e = s_pick[3];                   // pos_e >= 1: entry 0 is now, and E > 0
                const bool has_s = pos_s < n && __int_as_float(tl.e[pos_s].x) == S;
                const bool has_e = pos_e < n && __int_as_float(tl.e[pos_e].x) == E;
                const int occ_before_s = tl.e[pos_s > 0 ? pos_s - 1 : 0].y, occ_before_e = tl.e[pos_e - 1].y;
                const int old_len = hx_tl_len(2 * s_cnt[pd] - 1), new_len = hx_tl_len(2 * s_cnt[pd] + 1);
                __syncthreads();                                                  // every old entry has been read
                const int n_new = n + (has_s ? 0 : 1) + (has_e ? 0 : 1);
                if (in) {
                    const int at_new = tid + ((!has_s && tid >= pos_s) ? 1 : 0) + ((!has_e && tid >= pos_e) ? 1 : 0);
                    long long occ = me.y;
                    if (tid >= pos_s && tid < pos_e) occ += tok;
                    if (occ > (long long)INT_MAX) { hx_raise(a.status, HX_ERR_OVERFLOW); occ = INT_MAX; }
                    tl.e[at_new] = make_int2(me.x, (int)occ);
                }
                if (tid == 0 && !has_s) {
                    long long occ = (long long)occ_before_s + tok;
                    if (occ > (long long)INT_MAX) { hx_raise(a.status, HX_ERR_OVERFLOW); occ = INT_MAX; }
                    tl.e[pos_s] = make_int2(s_pick[4], (int)occ);
                }
                if (tid == HX_WAVE && !has_e) {
                    const int at_e = pos_e + (has_s ? 0 : 1);
                    tl.e[at_e] = make_int2(s_pick[5], occ_before_e);
                }
                // the filler behind the entries reaches as far as a timeline of two more events may be read
                for (int i = old_len + tid; i < new_len; i += DG_THREADS)
                    if (i >= n_new) tl.e[i] = make_int2(0x7f800000, 0);
                if (tid == 2 * HX_WAVE) s_n[pd] = n_new;
                __syncthreads();
            } else {
                hx_build_timeline<true>(s_cnt[pd], a.iv_start + at, a.iv_end + at, a.iv_tok + at, w, tl, &s_n[pd], a.status);
            }
            for (int c = tid; c < a.Q; c += DG_THREADS)
                if ((s_flags[c] & DG_ALIVE) && s_bd[c] == pd) s_flags[c] = DG_ALIVE | DG_DIRTY;
        }
        __syncthreads();
    }
    for (int d = tid; d < a.D; d += DG_THREADS) a.iv_count[d] = s_cnt[d];
}

// what a call has to know of an instance; the capacity stays an integer (as a float, some capacities are NaNs)
struct __align__(16) DPlanInst {
    float c1, c2, kB;
    int cap;
};

// LDS carve-up shared by host (size) and device (offsets)
struct DPlanLds {
    int ne, nt, D, Q;      // events per instance, stored timeline length, padded sizes
    __host__ __device__ DPlanLds(int stride, int D_, int Q_)
        : ne(2 * stride + 1), nt(hx_tl_len(2 * stride + 1) + 2), D((D_ + 3) & ~3), Q((Q_ + 3) & ~3) {}
    __host__ __device__ size_t off_red() const { return hx_align16((size_t)D * nt * 8); }                // int4 [2][2][wavefronts]
    __host__ __device__ size_t off_inst() const { return off_red() + 4 * 16 * (DP_MAX_THREADS / HX_WAVE); }    // DPlanInst per instance
    __host__ __device__ size_t off_n() const { return off_inst() + (size_t)16 * D; }                     // per instance: timeline entries, intervals
    __host__ __device__ size_t off_list() const { return off_n() + (size_t)8 * D; }                      // per slot: its call
    __host__ __device__ size_t off_call() const { return off_list() + (size_t)4 * Q; }                   // per call: L, O, lock, elapsed, tail, horizon, picked
    __host__ __device__ size_t off_scratch() const { return hx_align16(off_call() + (size_t)28 * Q); }
    __host__ __device__ size_t off_mat() const { return off_scratch() + hx_scratch_bytes(ne); }          // [D][Q] start of call c on instance d, +inf: none
    __host__ __device__ size_t bytes() const { return off_mat() + (size_t)D * Q * 4; }
};

// The plan where LDS has room for the start of every (instance, call) pair.  An added interval can only delay starts on
// the instance that received it, and there only those whose decode overlaps it: the calls of which this is true look
// for their start again, from where it was; a call whose best was there and moved takes the minimum of its row
// again (start + the call's decode time on the instance, the sum its finish was when the pair was scored).
//
// What bounds it: a pick is a chain of argmax, insertion into the timeline, scan and row minimum; a call is a lane, or
// several once the remaining calls leave lanes idle (their row is then split), the results of a call stay in its
// lanes' registers, every wavefront makes the pick for itself, the first one inserts.  Two barriers a pick.
// 256 calls on 32 instances 1350 -> 660 us, 100 on 32 500 -> 262, 1000 on 8 4530 -> 2650, 8 on 2 33 -> 26 (before: all 16
// wavefronts took part, one lane made the pick, every call looked again over the whole timeline).  Of 77 calls a pick that
// the new interval touches, nine move; the test against the most tokens held under it leaves few others.
// At most two lanes per call 687 us, four 662, eight 685; four wavefronts 737 instead of eight.
__global__ __launch_bounds__(DP_MAX_THREADS) void hx_decode_plan_kernel(DGreedyArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const DPlanLds lay(a.stride, a.D, a.Q);
    int2 *const s_tl = (int2 *)smem;
    int4 *const s_red = (int4 *)(smem + lay.off_red());
    DPlanInst *const s_inst = (DPlanInst *)(smem + lay.off_inst());
    int *const s_n = (int *)(smem + lay.off_n()), *const s_cnt = s_n + lay.D;
    int *const s_list = (int *)(smem + lay.off_list());
    int *const s_L = (int *)(smem + lay.off_call()), *const s_O = s_L + lay.Q, *const s_lk = s_O + lay.Q;
    float *const s_el = (float *)(s_lk + lay.Q), *const s_tail = s_el + lay.Q, *const s_hz = s_tail + lay.Q;
    int *const s_gone = (int *)(s_hz + lay.Q);
    float *const s_mat = (float *)(smem + lay.off_mat());
    __shared__ int s_wcnt[DP_MAX_THREADS / HX_WAVE], s_most;

    const int tid = threadIdx.x, NT = blockDim.x;
    const int lane = tid & (HX_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    for (int d = tid; d < a.D; d += NT) {
        int cnt = a.iv_count[d];
        if (cnt < 0 || cnt > a.stride) { hx_raise(a.status, HX_ERR_INDEX); cnt = cnt < 0 ? 0 : a.stride; }
        s_cnt[d] = cnt;
        const HxDecF x = hx_decode_terms(a.m, a.d_used[d], a.d_batch[d], 0, 1.0f / a.d_flops[d], 1.0f / a.d_hbm[d]);
        s_inst[d] = DPlanInst{x.c1, x.c2, x.kB, a.d_cap[d]};
    }
    for (int c = tid; c < a.Q; c += NT) {
        const int L = a.L_in[c], O = a.L_out[c], lk = a.lock ? a.lock[c] : -1;
        const bool fine = L >= 0 && O >= 0 && lk >= -1 && lk < a.D;      // otherwise the call has no place (lock -2)
        const int nd = a.node[c], w = a.wf[c];
        const bool ok = nd >= 0 && nd < a.n_nodes && w >= 0 && w < a.n_wf;
        if (!fine || !ok) hx_raise(a.status, HX_ERR_INDEX);
        s_L[c] = fine ? L : 0; s_O[c] = fine ? O : 0; s_lk[c] = fine ? lk : -2;
        s_el[c] = a.elapsed[c];
        s_tail[c] = ok ? a.tail[nd] : 0.0f;                    // tail of its node, horizon of its workflow (-1: index out of range)
        s_hz[c] = ok ? fmaxf(a.horizon[w], 0.0f) : -1.0f;
        s_gone[c] = 0;
        s_list[c] = c;
    }
    __syncthreads();
    // the timelines; the builders' scratch is where the matrix will be, as far as it goes
    const size_t one = hx_scratch_bytes(lay.ne);
    const int builders = min(NT / HX_WAVE, (int)((lay.bytes() - lay.off_scratch()) / one));
    int most = 0;
    for (int d = lane; d < a.D; d += HX_WAVE) most = max(most, s_cnt[d]);
    most = -hx_wave_min(-most);
    // An instance per wavefront, unless that leaves wavefronts without work (few instances, or scratch for few builders) over
    // lists that are long enough (an event is compared with every other): then one after the other by all of them.  Two
    // calls on 8 instances: lists of 10 23 us either way, 50 48 -> 30, 400 1235 -> 249; 256 calls on 32 with lists of 28 566
    // by a wavefront each and 620 by all.
    const long long n_ev = 2 * most + 1, rounds = (a.D + builders - 1) / builders;
    if (n_ev * n_ev * (rounds * NT - (long long)HX_WAVE * a.D) > (long long)DP_TOGETHER * a.D * HX_WAVE * NT) {
        for (int d = 0; d < a.D; ++d) {
            const size_t at = (size_t)d * a.stride;
            hx_build_timeline<false>(s_cnt[d], a.iv_start + at, a.iv_end + at, a.iv_tok + at,
                                     hx_carve_scratch(smem + lay.off_scratch(), lay.ne), Tl{s_tl + (size_t)d * lay.nt}, &s_n[d], a.status);
        }
    } else {
        for (int d = wave; d < a.D && wave < builders; d += builders) {
            const size_t at = (size_t)d * a.stride;
            hx_build_timeline<false, true>(s_cnt[d], a.iv_start + at, a.iv_end + at, a.iv_tok + at,
                                           hx_carve_scratch(smem + lay.off_scratch() + wave * one, lay.ne),
                                           Tl{s_tl + (size_t)d * lay.nt}, &s_n[d], a.status);
        }
    }
    __syncthreads();
    // tokens a call may find occupied on an instance, < 0: never fits, or has no place there
    auto threshold = [&](int L, int O, int lk, int d, int cap) {
        const long long room = (long long)cap - ((long long)L + (long long)O);
        return (room < 0 || (lk != -1 && lk != d)) ? -1 : (room > (long long)INT_MAX ? INT_MAX : (int)room);
    };
    // every start: a wavefront takes 64 calls on one instance at a time, all its lanes on the same timeline
    const int blocks = (a.Q + HX_WAVE - 1) / HX_WAVE;
    for (int i = wave; i < blocks * a.D; i += NT / HX_WAVE) {
        const int d = i / blocks, c = (i - d * blocks) * HX_WAVE + lane;
        const bool in = c < a.Q;
        const int L = in ? s_L[c] : 0, O = in ? s_O[c] : 0, lk = in ? s_lk[c] : -2;
        const DPlanInst x = s_inst[d];
        const HxSlot got = hx_earliest_start(s_tl + (size_t)d * lay.nt, s_n[d], threshold(L, O, lk, d, x.cap),
                                             hx_decode_time(hx_call_terms(a.m, L, O), x.c1, x.c2, x.kB), in);
        if (in) s_mat[d * lay.Q + c] = got.S;
    }
    __syncthreads();

    int n = a.Q, lanes = NT;
    for (int k = 0; k < a.Q;) {
        // ---- a stage: the remaining calls in increasing order, G lanes each; a wavefront per 64 lanes
        const int n_before = n;
        n = a.Q - k;
        if (k > 0) {
            const int c = s_list[tid < n_before ? tid : 0];
            const bool stays = tid < n_before && s_gone[c] == 0;
            const u64 b = __builtin_amdgcn_ballot_w64(stays);
            if (lane == 0) s_wcnt[wave] = __popcll(b);
            __syncthreads();
            int at = __popcll(b & ((1ull << lane) - 1ull));
            for (int v = 0; v < wave; ++v) at += s_wcnt[v];
            if (stays) s_list[at] = c;
            __syncthreads();
        }
        int lg = 0;
        while ((2 << lg) <= DP_MAX_G && (n << (lg + 1)) <= lanes) ++lg;
        const int G = 1 << lg, n_lanes = n << lg, n_waves = (n_lanes + HX_WAVE - 1) / HX_WAVE;
        lanes = n_waves * HX_WAVE;
        const int last = n_waves > 1 ? a.Q - n / 2 : a.Q;      // the stage's picks end here
        const int slot = tid >> lg, sub = tid & (G - 1);
        bool alive = slot < n;
        const int c = s_list[alive ? slot : 0];                // lanes without a call go along with the first one's and write nothing
        const int L = s_L[c], O = s_O[c], lk = s_lk[c];
        const float el = s_el[c], tail = s_tail[c], hz = s_hz[c];
        const HxCallF cf = hx_call_terms(a.m, L, O);
        float best = INFINITY;
        int best_d = INT_MAX;
        unsigned ratio_bits = 0;
        // the earliest finish of the lane's call, the lowest instance that has it, and its ratio, Eq. (2)
        auto row = [&]() {
            float v = INFINITY;
            int at = INT_MAX;
#pragma unroll 4
            for (int d = sub; d < a.D; d += G) {               // ascending, strictly smaller
                const DPlanInst x = s_inst[d];
                const float f = s_mat[d * lay.Q + c] + hx_decode_time(cf, x.c1, x.c2, x.kB);
                at = f < v ? d : at;
                v = fminf(v, f);
            }
            best = hx_lanes_min(v, G);
            best_d = hx_lanes_min(v == best ? at : INT_MAX, G);
            ratio_bits = hx_ratio_bits(el, best, tail, hz, hz >= 0.0f);
        };
        if (wave < n_waves) row();
        if (wave >= n_waves) {                                 // no calls here any more
            if (n_waves > 1)
                for (int i = k; i < last; ++i) { __syncthreads(); __syncthreads(); }
            k = last;
        }
        for (; k < last; ++k) {
            // (1) the most urgent remaining call: largest ratio, lowest index among equals (slots, and with them lanes and
            // wavefronts, are in index order)
            const float key = alive ? hx_rank_key(ratio_bits) : -INFINITY;
            const float top = hx_wave_max(key);
            const u64 at_top = __builtin_amdgcn_ballot_w64(alive && key == top);
            int from = at_top ? __builtin_ctzll(at_top) : 0;   // (no lane with a call: it loses to every wavefront that has one)
            int pick = at_top ? (wave * HX_WAVE + from) >> lg : INT_MAX;
            int pc = __builtin_amdgcn_readlane(c, from), pd = __builtin_amdgcn_readlane(best_d, from);
            float E = hx_lane_value(best, from);
            int p_ratio = __builtin_amdgcn_readlane((int)ratio_bits, from);
            if (n_waves > 1) {
                int4 *red = s_red + (k & 1) * 2 * (DP_MAX_THREADS / HX_WAVE);
                if (lane == 0) {
                    red[wave] = make_int4(__float_as_int(top), pick, pc, pd);
                    red[DP_MAX_THREADS / HX_WAVE + wave] = make_int4(__float_as_int(E), p_ratio, 0, 0);
                }
                __syncthreads();
                const int v = min(lane, n_waves - 1);          // (n_waves is at most a row of lanes; lanes beyond repeat the last)
                const int4 q = red[v], q2 = red[DP_MAX_THREADS / HX_WAVE + v];
                const float all = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(-hx_lanes_min(-__int_as_float(q.x), n_waves))));
                from = __builtin_ctzll(__builtin_amdgcn_ballot_w64(q.y != INT_MAX && __int_as_float(q.x) == all));
                pick = __builtin_amdgcn_readlane(q.y, from);
                pc = __builtin_amdgcn_readlane(q.z, from); pd = __builtin_amdgcn_readlane(q.w, from);
                E = __int_as_float(__builtin_amdgcn_readlane(q2.x, from)); p_ratio = __builtin_amdgcn_readlane(q2.y, from);
            }
            const bool placed = pd != INT_MAX;
            const float S = placed ? s_mat[pd * lay.Q + pc] : INFINITY;
            const int cnt = placed ? s_cnt[pd] : 0, n_old = placed ? s_n[pd] : 1;
            const bool added = placed && cnt < a.stride;
            const long long need = placed ? (long long)s_L[pc] + (long long)s_O[pc] : 0;
            const int tok = need > (long long)INT_MAX ? INT_MAX : (int)need;
            // An interval that holds nothing (a call without output tokens) leaves the timeline as it is, and nobody has to look
            // again: 1000 calls on 8 instances with lists of 428, a third of them such calls, 10.8 -> 3.6 ms (the first
            // wavefront built the timeline again for each).  Any other one starts now or later and, as its call was
            // placed, ends at a finite time: it is inserted.
            const bool nothing = !(S < E) || need <= 0;
            alive = alive && slot != pick;
            int2 *const tl = s_tl + (added ? pd : 0) * lay.nt;
            // (2) the first wavefront adds its interval (the last one records the pick)
            const size_t at = (size_t)(added ? pd : 0) * a.stride + cnt;
            if (wave == n_waves - 1 && lane == 0) {
                a.best_d[pc] = placed ? pd : -1; a.best_start[pc] = S; a.best_cost[pc] = E; a.rank[pc] = k;
                hx_store_bits(a.ratio, pc, (unsigned)p_ratio);
                s_gone[pc] = 1;
                if (placed && !added) hx_raise(a.status, HX_ERR_CAPACITY);
                if (added) { a.iv_start[at] = S; a.iv_end[at] = E; a.iv_tok[at] = tok; }
            }
            if (wave == 0) {
                // the filler behind the n entries reaches as far as a timeline of two more events may be read
                auto fill = [&](int n_tl) {
                    const int i = hx_tl_len(2 * cnt + 1) + lane;
                    if (i < hx_tl_len(2 * cnt + 3) && i >= n_tl) tl[i] = make_int2(0x7f800000, 0);
                };
                if (added && !nothing) {
                    // The compact timeline is a function of the instance's events, so adding the two events of the new
                    // interval (S, E, tok) to it gives what building it again would: entries from S up to E hold tok
                    // more; S and E become entries of their own unless the timeline already has an entry at that time
                    // (S: the occupancy before it plus tok; E: the occupancy that stood before E).
                    int pos_s = 0, pos_e = 0;
                    bool has_s = false, has_e = false;
                    const int top0 = (n_old - 1) & ~(HX_WAVE - 1);
                    const int2 tail_me = tl[min(top0 + lane, n_old - 1)];      // of the last 64 entries
                    if (top0 == 0) {
                        const float t = lane < n_old ? __int_as_float(tail_me.x) : INFINITY;      // S and E are finite
                        pos_s = __popcll(__builtin_amdgcn_ballot_w64(t < S)); pos_e = __popcll(__builtin_amdgcn_ballot_w64(t < E));
                        has_s = __builtin_amdgcn_ballot_w64(t == S) != 0; has_e = __builtin_amdgcn_ballot_w64(t == E) != 0;
                    } else {
                        // more than 64 entries: every seg-th first, then the seg of them (at most 16) that lead up to the place, by
                        // half a wavefront for S and the other for E
                        const int seg = (n_old + HX_WAVE - 1) / HX_WAVE;
                        const float t = lane * seg < n_old ? __int_as_float(tl[lane * seg].x) : INFINITY;
                        const int from_s = max((int)__popcll(__builtin_amdgcn_ballot_w64(t < S)) - 1, 0) * seg;
                        const int from_e = max((int)__popcll(__builtin_amdgcn_ballot_w64(t < E)) - 1, 0) * seg;
                        const int i = (lane < 32 ? from_s : from_e) + (lane & 31);
                        const bool in = (lane & 31) <= seg && i < n_old;      // (one more: the entry at the place itself)
                        const float u = in ? __int_as_float(tl[i].x) : INFINITY, mine = lane < 32 ? S : E;
                        const u64 before = __builtin_amdgcn_ballot_w64(u < mine), same = __builtin_amdgcn_ballot_w64(u == mine);
                        pos_s = from_s + (int)__popc((unsigned)before); pos_e = from_e + (int)__popc((unsigned)(before >> 32));
                        has_s = (unsigned)same != 0; has_e = (unsigned)(same >> 32) != 0;
                    }
                    int2 me = tail_me;
                    // pos_e >= 1: entry 0 is now, and E > 0
                    const int before_s = max(pos_s - 1, 0), before_e = pos_e - 1;
                    const int occ_before_s = top0 == 0 ? __builtin_amdgcn_readlane(me.y, before_s) : tl[before_s].y;
                    const int occ_before_e = top0 == 0 ? __builtin_amdgcn_readlane(me.y, before_e) : tl[before_e].y;
                    bool over = false;
                    int most = 0;                              // tokens held at most from S up to E
                    auto more = [&](int occ) {
                        const int sum = __builtin_elementwise_add_sat(occ, tok);      // both are >= 0
                        over = over || sum - occ != tok;
                        most = max(most, sum);
                        return sum;
                    };
                    // from the last 64 entries to those at S: an entry moves by two places at most, towards the end
                    for (int i0 = top0; i0 >= 0 && i0 + HX_WAVE > pos_s; i0 -= HX_WAVE) {
                        const int i = i0 + lane;
                        if (i0 != top0) me = tl[i];
                        hx_wave_sync();
                        if (i < n_old)
                            tl[i + (!has_s && i >= pos_s) + (!has_e && i >= pos_e)] = make_int2(me.x, i >= pos_s && i < pos_e ? more(me.y) : me.y);
                        hx_wave_sync();
                    }
                    const int n_new = n_old + !has_s + !has_e;
                    if (lane == 0) {
                        if (!has_s) tl[pos_s] = make_int2(__float_as_int(S > 0.0f ? S : 0.0f), more(occ_before_s));
                        if (!has_e) tl[pos_e + !has_s] = make_int2(__float_as_int(E), occ_before_e);
                        s_n[pd] = n_new;
                    }
                    most = -hx_wave_min(-most);
                    if (lane == 0) s_most = most;
                    if (over) hx_raise(a.status, HX_ERR_OVERFLOW);
                    fill(n_new);
                } else if (added) {
                    fill(n_old);
                }
                hx_wave_sync();
            }
            if (n_waves > 1) __syncthreads();
            if (!added) continue;
            if (tid == 0) s_cnt[pd] = cnt + 1;                 // (every wavefront has read it)
            if (nothing) continue;
            // (3) who has to look again: where the call may go at all, if its start with its decode time touches the new
            // interval, and some moment of that leaves it no room.  A start needs room at its own moment, however short
            // the decode time (0, or lost in the addition): S <= old stands beside the window's S < old + T.
            const DPlanInst x = s_inst[pd];
            const float T = hx_decode_time(cf, x.c1, x.c2, x.kB);
            const int thr = threshold(L, O, lk, pd, x.cap);
            const float old = s_mat[pd * lay.Q + c];
            const bool touched = alive && sub == 0 && old < INFINITY && old < E && (S <= old || S < old + T) && thr < s_most;
            u64 todo = __builtin_amdgcn_ballot_w64(touched);
            if (todo == 0) continue;
            const int n_tl = s_n[pd];
            float now = INFINITY;
            if (n_tl <= HX_WAVE && __popcll(todo) <= DP_FEW) {
                // Few calls on a timeline of few entries: one call after the other, a lane per entry.  An entry where
                // a run of entries with room begins is a start if the run's end, the next entry without, is far enough.
                const int2 me = tl[lane];                      // behind the last entry: never, empty
                const float t = __int_as_float(me.x);
                while (todo) {
                    const int ld = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    const u64 full = __builtin_amdgcn_ballot_w64(lane < n_tl && me.y > __builtin_amdgcn_readlane(thr, ld));
                    const float T_ld = hx_lane_value(T, ld);
                    u64 runs = ~full & ((full << 1) | 1);      // first entries of the runs
                    float got = INFINITY;
                    while (runs) {
                        const int i = __builtin_ctzll(runs);
                        const u64 end = full >> i;
                        const float rs = hx_lane_value(t, i), re = end ? hx_lane_value(t, i + __builtin_ctzll(end)) : INFINITY;
                        if (i >= n_tl) break;
                        if (re >= rs + T_ld) { got = rs; break; }
                        runs &= runs - 1;
                    }
                    now = lane == ld ? got : now;
                }
            } else {
                // its start was the earliest, and load was only added: nothing before it can be one now
                int begin = 0;
                for (int i0 = 8; i0 < n_tl; i0 += 64) {
                    float t[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) t[u] = __int_as_float(tl[min(i0 + 8 * u, n_tl)].x);      // entry n: never
#pragma unroll
                    for (int u = 0; u < 8; ++u) begin += touched && t[u] <= old ? 8 : 0;
                }
                now = hx_earliest_start(tl, n_tl, thr, T, touched, begin).S;
            }
            if (touched) s_mat[pd * lay.Q + c] = now;
            const u64 moved = __builtin_amdgcn_ballot_w64(touched && best_d == pd && now != old);
            hx_wave_sync();
            if (moved) row();
        }
        __syncthreads();
    }
    for (int d = tid; d < a.D; d += NT) a.iv_count[d] = s_cnt[d];
}

__global__ __launch_bounds__(256) void hx_decode_no_instance_kernel(DGreedyArgs a)
{
    // no decode instance at all: nothing is feasible, every call has infinite ratio and is ranked by index
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.Q) return;
    a.best_d[c] = -1; a.best_start[c] = INFINITY; a.best_cost[c] = INFINITY; a.rank[c] = c;
    hx_projected_ratio(a.node, a.wf, a.elapsed, a.tail, a.horizon, a.n_nodes, a.n_wf, c, INFINITY, a.status, a.ratio);
}

HxModelF to_model(const hx_model *m)
{
    return HxModelF{m->kv_bytes_per_token, m->flops_per_token, m->attn_flops_per_token2, m->weight_bytes, m->nominal_batch};
}

int check_tables(hx_ctx *ctx, const hx_calls *q, const hx_decode_tab *dec, const hx_intervals *iv)
{
    HX_REQUIRE(ctx, q->n >= 0 && dec->n >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, dec->n <= HX_MAX_INSTANCES, HX_ERR_SHAPE, "%d decode instances, at most %d", dec->n, HX_MAX_INSTANCES);
    HX_REQUIRE(ctx, iv->stride >= 0 && iv->stride <= HX_MAX_INTERVALS, HX_ERR_SHAPE,
               "interval stride %d outside 0..%d", iv->stride, HX_MAX_INTERVALS);
    HX_REQUIRE(ctx, q->n == 0 || (q->L_in && q->L_out), HX_ERR_INVALID_ARG, "NULL call lengths");
    HX_REQUIRE(ctx, dec->n == 0 || (dec->flops && dec->hbm_bw && dec->used_tok && dec->cap_tok && dec->batch && iv->count),
               HX_ERR_INVALID_ARG, "NULL decode table or interval count");
    HX_REQUIRE(ctx, dec->n == 0 || iv->stride == 0 || (iv->start && iv->end && iv->tok), HX_ERR_INVALID_ARG, "NULL interval array");
    return HX_OK;
}

}  // namespace

// the decode planners may use all of a CU's LDS; said once per process
constexpr size_t DP_LDS = 160 * 1024 - 128;                  // but for the first one's own counters
int hx_decode_init()
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(hx_decode_plan_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, DP_LDS);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(hx_decode_plan_lean_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    return e == hipSuccess ? HX_OK : HX_ERR_DEVICE;
}

extern "C" int hx_decode_score(hx_ctx *ctx, const hx_model *model, const hx_calls *queue, const int32_t *lock,
                               const hx_decode_tab *dec, const hx_intervals *iv,
                               const float *tail, const float *horizon, int32_t n_nodes, int32_t n_wf,
                               float *start, float *cost,
                               int32_t *best_d, float *best_start, float *best_cost, float *ratio, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HX_REQUIRE(ctx, model && queue && dec && iv, HX_ERR_INVALID_ARG, "NULL table");
    if (int rc = check_tables(ctx, queue, dec, iv)) return rc;
    const int Q = queue->n, D = dec->n;
    HX_REQUIRE(ctx, Q == 0 || (best_d && best_start && best_cost), HX_ERR_INVALID_ARG, "NULL output");
    HX_REQUIRE(ctx, !ratio || Q == 0 || (queue->node && queue->wf && queue->elapsed && tail && horizon), HX_ERR_INVALID_ARG,
               "a ratio needs node, wf, elapsed, tail and horizon");
    HX_REQUIRE(ctx, n_nodes >= 0 && n_wf >= 0, HX_ERR_INVALID_ARG, "negative n_nodes or n_wf");
    if (Q == 0) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;
    const int ne = 2 * iv->stride + 1, nt = hx_tl_len(ne);
    // Without the pairs' matrices only the best instance of a call is wanted, which few pairs decide.
    const bool pairs = start || cost;
    // Groups of instances: enough workgroups (tiles of 256 calls x groups) to fill the chip several times over,
    // at most 64 groups (the finish kernel reads one partial result per group and call).
    const int tiles = (Q + DS_THREADS - 1) / DS_THREADS;
    int n_groups = 0, gd = 1;
    if (D > 0 && pairs) {
        n_groups = (8 * ctx->num_cu + tiles - 1) / tiles;
        if (n_groups > 64) n_groups = 64;
        if (n_groups > D) n_groups = D;
        gd = (D + n_groups - 1) / n_groups;
        n_groups = (D + gd - 1) / gd;
    }
    const int per = D > 0 ? (Q + D - 1) / D : Q;
    // words of scratch per pass: the free list (D slices of `per` places) and three partial results per group and call
    const size_t part_need = pairs && D > 0 ? (size_t)D * per + 3 * (size_t)n_groups * Q : 0;
    const size_t tl_need = (size_t)(D > 0 ? D : 1) * nt;
    const int tab_need = pairs ? D : 0;
    if (part_need > ctx->dpart_cap || tl_need > ctx->dtl_cap || tab_need > ctx->dtab_cap) {
        // grown, never shrunk; work queued on the old blocks has to finish before they go
        HX_HIP(ctx, hipDeviceSynchronize());
        if (part_need > ctx->dpart_cap) {
            if (ctx->d_dpart) { HX_HIP(ctx, hipFree(ctx->d_dpart)); ctx->d_dpart = nullptr; ctx->dpart_cap = 0; }
            const size_t want = part_need < 65536 ? 65536 : part_need;
            HX_HIP(ctx, hipMalloc((void **)&ctx->d_dpart, want * sizeof(int32_t)));
            ctx->dpart_cap = want;
        }
        if (tl_need > ctx->dtl_cap) {
            if (ctx->d_dtl) { HX_HIP(ctx, hipFree(ctx->d_dtl)); ctx->d_dtl = nullptr; ctx->dtl_cap = 0; }
            // per entry: (time, occupancy) and (head time, head rank) 8 bytes each, sorted occupancy and stretch head 4
            // each, source 2; per instance two counts and a record of eight words
            HX_HIP(ctx, hipMalloc((void **)&ctx->d_dtl, tl_need * 24 + (2 + 8) * (size_t)HX_MAX_INSTANCES * sizeof(int) + 64));
            ctx->dtl_cap = tl_need;
        }
        if (tab_need > ctx->dtab_cap) {
            if (ctx->d_dtab) { HX_HIP(ctx, hipFree(ctx->d_dtab)); ctx->d_dtab = nullptr; ctx->dtab_cap = 0; }
            const int want = D < 64 ? 64 : D;
            HX_HIP(ctx, hipMalloc((void **)&ctx->d_dtab, (size_t)want * HX_TAB * sizeof(float)));
            ctx->dtab_cap = want;
        }
    }
    TlOut o{};
    int32_t *n_free = nullptr;
    {
        unsigned char *p = (unsigned char *)ctx->d_dtl;
        const size_t cap = ctx->dtl_cap;                      // a multiple of 8: every block below stays 16-byte aligned
        o.e = (int2 *)p;        p += cap * 8;
        o.head = (int2 *)p;     p += cap * 8;
        o.n = (int *)p;         p += (size_t)HX_MAX_INSTANCES * sizeof(int);
        n_free = (int32_t *)p;  p += (size_t)HX_MAX_INSTANCES * sizeof(int);
        o.meta = (int *)p;      p += 8 * (size_t)HX_MAX_INSTANCES * sizeof(int);
        o.sorted = (int *)p;    o.least = o.sorted;    p += cap * 4;
        o.seg = (int *)p;       o.step = o.seg;    p += cap * 4;
        o.G = ctx->d_dtab;
    }
    int32_t *free_c = ctx->d_dpart;
    float *part_cost = (float *)(ctx->d_dpart + (size_t)D * per);
    float *part_start = part_cost + (size_t)n_groups * Q;
    int32_t *part_d = (int32_t *)(part_start + (size_t)n_groups * Q);
    DecodeFinishArgs f{};
    f.Q = Q; f.D = D; f.n_groups = n_groups;
    f.L_in = queue->L_in; f.L_out = queue->L_out; f.lock = lock;
    f.part_cost = part_cost; f.part_start = part_start; f.part_d = part_d;
    f.node = queue->node; f.wf = queue->wf; f.elapsed = queue->elapsed; f.tail = tail; f.horizon = horizon;
    f.n_nodes = n_nodes; f.n_wf = n_wf;
    f.best_d = best_d; f.best_start = best_start; f.best_cost = best_cost; f.ratio = ratio; f.status = ctx->d_status;
    if (D > 0) {
        DecodeArgs a{};
        a.m = to_model(model); a.Q = Q; a.D = D; a.stride = iv->stride;
        a.L_in = queue->L_in; a.L_out = queue->L_out; a.lock = lock;
        a.d_flops = dec->flops; a.d_hbm = dec->hbm_bw; a.d_used = dec->used_tok; a.d_cap = dec->cap_tok; a.d_batch = dec->batch;
        a.iv_count = iv->count; a.iv_start = iv->start; a.iv_end = iv->end; a.iv_tok = iv->tok;
        a.start = start; a.cost = cost; a.status = ctx->d_status;
        a.free_c = free_c; a.n_free = n_free; a.per = per;
        a.gd = gd; a.n_groups = n_groups; a.part_cost = part_cost; a.part_start = part_start; a.part_d = part_d;
        if (!pairs) {
            a.tries = DB_TRIES / D < 1 ? 1 : (DB_TRIES / D < DO_THREADS / HX_WAVE - 1 ? DB_TRIES / D : DO_THREADS / HX_WAVE - 1);
            const int n_tries = a.tries * D;
            a.try_step = Q / n_tries > 1 ? Q / n_tries : 1;
            a.try_mask = INT_MAX;
            while (n_tries * a.try_step > Q && a.try_mask >= Q) a.try_mask >>= 1;       // fewer calls than tries
            hx_decode_occupancy_kernel<<<D, DO_THREADS, 0, stream>>>(a, o, nt);
            // a wavefront per call, and workgroups with a place of their own as long as there are
            const int waves = DB_THREADS / HX_WAVE, most = DB_PER_CU * ctx->num_cu, few = 2 * ctx->num_cu;
            int grid = Q / waves + (Q % waves != 0);
            grid = grid < few ? (Q < few ? Q : few) : (grid < most ? grid : most);
            // where every pair is formed, calls a workgroup takes together: as many workgroups as there are places for (16384 calls on 256 instances
            // in pieces: 16 79 us, 4 90; 4000: 16 39, 4 30; 300 on 1024: 4 64, 1 46)
            const int G = Q > waves * most ? 16 : (Q > few ? 4 : 1);
            if (D <= HX_WAVE) hx_decode_best_kernel<1><<<grid, DB_THREADS, 0, stream>>>(a, f, o, nt, G);
            else if (D <= 4 * HX_WAVE) hx_decode_best_kernel<4><<<grid, DB_THREADS, 0, stream>>>(a, f, o, nt, G);
            else if (D <= 8 * HX_WAVE) hx_decode_best_kernel<8><<<grid, DB_THREADS, 0, stream>>>(a, f, o, nt, G);
            else hx_decode_best_kernel<HX_MAX_INSTANCES / HX_WAVE><<<grid, DB_THREADS, 0, stream>>>(a, f, o, nt, G);
            return hx_check_launch(ctx, "hx_decode_score kernels");
        }
        const size_t lds = hx_scratch_bytes(ne) + hx_align16((size_t)nt * 8);
        hx_decode_timeline_kernel<<<D, TL_THREADS, lds, stream>>>(a, o, nt);
        const int n_lock = lock ? tiles : 0;
        hx_decode_score_kernel<<<n_lock + tiles * n_groups, DS_THREADS, 0, stream>>>(a, o, nt, n_lock);
    }
    hx_decode_finish_kernel<<<(Q + 63) / 64, 64, 0, stream>>>(f);
    return hx_check_launch(ctx, "hx_decode_score kernels");
}

// whether a shape's plan is made without the start of every pair (tests ask too)
extern "C" int hx_test_decode_plan_lean(int stride, int D, int Q) { return DPlanLds(stride, D, Q).bytes() > DP_LDS; }

extern "C" int hx_decode_plan_greedy(hx_ctx *ctx, const hx_model *model, const hx_calls *queue, const int32_t *lock,
                                     const hx_decode_tab *dec, const hx_intervals *iv,
                                     const float *tail, const float *horizon, int32_t n_nodes, int32_t n_wf,
                                     int32_t *best_d, float *best_start, float *best_cost, float *ratio, int32_t *rank,
                                     void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HX_REQUIRE(ctx, model && queue && dec && iv, HX_ERR_INVALID_ARG, "NULL table");
    if (int rc = check_tables(ctx, queue, dec, iv)) return rc;
    const int Q = queue->n, D = dec->n;
    HX_REQUIRE(ctx, Q <= HX_DECODE_GREEDY_MAX_CALLS, HX_ERR_SHAPE, "%d calls beyond the %d the decode planner takes", Q,
               HX_DECODE_GREEDY_MAX_CALLS);
    HX_REQUIRE(ctx, Q == 0 || (best_d && best_start && best_cost && ratio && rank), HX_ERR_INVALID_ARG, "NULL output");
    HX_REQUIRE(ctx, Q == 0 || (queue->node && queue->wf && queue->elapsed && tail && horizon), HX_ERR_INVALID_ARG,
               "the planner needs node, wf, elapsed, tail and horizon");
    HX_REQUIRE(ctx, n_nodes >= 0 && n_wf >= 0, HX_ERR_INVALID_ARG, "negative n_nodes or n_wf");
    if (Q == 0) return HX_OK;
    const DGreedyLds lay(iv->stride, D, Q);
    HX_REQUIRE(ctx, lay.bytes() <= (size_t)160 * 1024, HX_ERR_SHAPE,
               "%d instances x %d entries (+ %d calls) need %zu bytes of local memory, at most %d", D, iv->stride, Q,
               lay.bytes(), 160 * 1024);
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;
    DGreedyArgs a{};
    a.m = to_model(model); a.Q = Q; a.D = D; a.stride = iv->stride;
    a.L_in = queue->L_in; a.L_out = queue->L_out; a.lock = lock; a.node = queue->node; a.wf = queue->wf;
    a.elapsed = queue->elapsed; a.tail = tail; a.horizon = horizon; a.n_nodes = n_nodes; a.n_wf = n_wf;
    a.d_flops = dec->flops; a.d_hbm = dec->hbm_bw; a.d_used = dec->used_tok; a.d_cap = dec->cap_tok; a.d_batch = dec->batch;
    a.iv_count = iv->count; a.iv_start = iv->start; a.iv_end = iv->end; a.iv_tok = iv->tok;
    a.best_d = best_d; a.best_start = best_start; a.best_cost = best_cost; a.ratio = ratio; a.rank = rank;
    a.status = ctx->d_status;
    if (D == 0) {
        hx_decode_no_instance_kernel<<<(Q + 255) / 256, 256, 0, stream>>>(a);
    } else {
        const size_t lds = DPlanLds(iv->stride, D, Q).bytes();
        // The widest workgroup also where few calls meet long lists: the calls need no more lanes, but the timelines are built by all
        // of them (64 calls on 8 instances with lists of 310: 592 -> 532 us; 200 calls, which would be dealt to more lanes: 1452 ->
        // 1577; lists of 128 and fewer: no difference).
        const bool wide = Q > DP_THREADS || (Q * DP_MAX_G <= DP_THREADS && iv->stride >= 256);
        if (!hx_test_decode_plan_lean(iv->stride, D, Q)) hx_decode_plan_kernel<<<1, wide ? DP_MAX_THREADS : DP_THREADS, lds, stream>>>(a);
        else hx_decode_plan_lean_kernel<<<1, DG_THREADS, lay.bytes(), stream>>>(a);
    }
    return hx_check_launch(ctx, "hx_decode_plan_greedy kernel");
}
