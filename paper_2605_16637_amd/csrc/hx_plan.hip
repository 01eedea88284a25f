// The planner around the scoring loop (Algorithm 1 main loop; Sec. 5.3):
// one-pass ordering of the calls by their projected ratio, and the recomputing
// greedy loop for small queues -- pick the most urgent call, give it the pair
// with the earliest projected decode finish, add it to a simulated copy of the
// pool state, score again.
#include "hx_common.hpp"
#include "hx_terms.hpp"
#include "hx_search.hpp"

#include <cmath>
#include <cstdlib>
#include <type_traits>

namespace {

constexpr int kT = HX_MAX_TYPES;

// ---- one-pass ordering -----------------------------------------------------------

constexpr int RANK_TILE = 2048;      // calls compared against per block, at most
constexpr int RANK_PAIRS = 10 * 1024;     // queues up to this size are ranked by all-pairs counting

__global__ __launch_bounds__(256) void hx_rank_zero_kernel(int32_t *rank, int C)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < C) rank[c] = 0;
}

// (ratio, index) as one unsigned 64-bit key that orders like "larger ratio first,
// then lower index": the float bits made monotone, then the complemented index
__device__ __forceinline__ unsigned long long hx_rank_key64(unsigned bits, int idx)
{
    unsigned b = __float_as_uint(hx_rank_key(bits));
    b ^= (b & 0x80000000u) ? 0xffffffffu : 0x80000000u;
    return ((unsigned long long)b << 32) | (unsigned)(0xffffffffu - (unsigned)idx);
}

// rank[c] = number of calls ahead of c: larger ratio, or equal ratio and lower index.  Short queues: a workgroup ranks 64
// calls, a lane each, its wavefronts comparing them with a share of the queue each; one launch, nothing to
// clear.  Launches back to back, two of them before and one now: 64 calls 4.7 -> 3.1 us, 1024 5.3 -> 4.8; 1200 5.2 either
// way, 2048 would be 7.1 instead of 5.6.
constexpr int RANK_THREADS = 1024;
constexpr int RANK_DIRECT = 1024;

__global__ __launch_bounds__(RANK_THREADS) void hx_rank_direct_kernel(const float *ratio, int32_t *rank, int C)
{
    __shared__ unsigned long long s_key[RANK_DIRECT];
    __shared__ int s_ahead[HX_WAVE];
    const int tid = threadIdx.x, lane = tid & (HX_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.x * HX_WAVE + lane;
    for (int i = tid; i < C; i += RANK_THREADS) s_key[i] = hx_rank_key64(hx_load_bits(ratio, i), i);
    if (tid < HX_WAVE) s_ahead[tid] = 0;
    __syncthreads();
    const unsigned long long mine = s_key[min(c, C - 1)];
    const int share = (C + RANK_THREADS / HX_WAVE - 1) / (RANK_THREADS / HX_WAVE);
    const int end = min((wave + 1) * share, C);
    int ahead = 0;
#pragma unroll 8
    for (int i = wave * share; i < end; ++i) ahead += s_key[i] > mine;
    if (ahead) atomicAdd(&s_ahead[lane], ahead);
    __syncthreads();
    if (tid < HX_WAVE && c < C) rank[c] = s_ahead[tid];
}

// Longer queues, up to RANK_PAIRS: rank[c] = number of calls ahead of c: larger ratio, or equal ratio and lower
// index.  Block (i, j) counts, for 256 calls, those ahead of them among the
// `tile` calls of tile j; the partial counts are added up with integer atomics.
__global__ __launch_bounds__(256) void hx_rank_count_kernel(const float *ratio, int32_t *rank, int C, int tile)
{
    __shared__ unsigned long long s_key[RANK_TILE];
    const int k0 = blockIdx.y * tile;
    const int kn = min(tile, C - k0);
    for (int i = threadIdx.x; i < kn; i += blockDim.x) s_key[i] = hx_rank_key64(hx_load_bits(ratio, k0 + i), k0 + i);
    __syncthreads();
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    const unsigned long long mine = hx_rank_key64(hx_load_bits(ratio, c), c);
    int ahead = 0;
#pragma unroll 8
    for (int i = 0; i < kn; ++i) ahead += s_key[i] > mine;
    if (ahead) atomicAdd(&rank[c], ahead);
}

// Beyond RANK_PAIRS calls, up to RANK_CUT: one launch of a workgroup per bucket.  RANK_CUTS calls, one from each of as
// many stretches of the queue and anywhere in it, are ordered by counting; workgroup b takes the calls between the b-th of
// them and the next.  It reads the whole queue, counts the calls ahead of its bucket, gathers the bucket's members in LDS and counts among those.  Keys
// are unique (they end in the call index), so the buckets stay balanced however many ratios are equal.  Up to RANK_BY_PAIRS members
// are compared with each other, more are sorted; should they outgrow the LDS, the queue is sorted a part at a time (what is not of the
// bucket at the end) and every member's place looked up in each.
// Bound: two round trips and the ordering of the cuts (7 us together), then the pass over the queue and the largest bucket,
// some six times the others (it differs from queue to queue).  Launches back to back, random ratios, all pairs of calls / cuts / the sample
// sort below: 10241 calls 13.3 / 12 (10 to 14) / -, 12000 15.1 / 12.7 (up to 14.5) / -, 16384 22.4 / 14.3 (up to 18.9) / -, 24000 - / 18.7 (up
// to 25) / 23 to 35, 28000 - / 22.8 (up to 26.6) / 25 to 35.  Members of one bucket among 16384 calls, by pairs and sorted: 300 10.5 and -, 500 12.1
// and 19, 700 17.0 and 19.7, 800 22.1 and 20.0, 1000 25 and 20, 4000 - and 43 (by pairs 64 members at a time, with two barriers each: 500
// 16.0, 700 23).  A queue whose dividers all lie above the other calls: 168 us of 10241 calls, 275 of 16384, 640 of 28672, the
// lookups, whose LDS reads lie anywhere, two thirds of it (members counted against the whole queue by pairs: 7 to 57 ms).
// (Cuts compared as 32-bit words with the ties by index, four at a time: 1.5 us more; workgroups of 512 threads: 0.5
// less on 2048 calls, 3 more on 16384.)
constexpr int RANK_CUT = 28 * 1024;
constexpr int RANK_CUTS = 255;                   // buckets 0 .. RANK_CUTS
constexpr int RANK_MEMBERS = 4096;               // members of a bucket that LDS holds (a power of two)
constexpr int RANK_BY_PAIRS = 768;               // members compared with each other
constexpr int RANK_GROUPS = 4;                   // of 64 members, in flight together
constexpr int RANK_READ = 8;                     // calls a thread has in flight

__global__ __launch_bounds__(RANK_THREADS) void hx_rank_cut_kernel(const float *ratio, int32_t *rank, int C)
{
    __shared__ unsigned long long s_cut[RANK_CUTS + 1], s_key[RANK_MEMBERS], s_low, s_high;
    __shared__ int s_place[RANK_CUTS + 1], s_higher, s_n, s_ahead[RANK_BY_PAIRS];
    const int tid = threadIdx.x, lane = tid & (HX_WAVE - 1), b = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int WAVES = RANK_THREADS / HX_WAVE;
    if (tid <= RANK_CUTS) {
        // call of stretch tid (a multiplicative hash says where in it; the queue holds more calls than there are stretches)
        const long long begin = (long long)tid * C / (RANK_CUTS + 1), size = (long long)(tid + 1) * C / (RANK_CUTS + 1) - begin;
        const int c = (int)(begin + (((unsigned)tid * 2654435761u >> 8) * (unsigned long long)size >> 24));
        s_cut[tid] = tid < RANK_CUTS ? hx_rank_key64(hx_load_bits(ratio, c), c) : 0ull;
        s_place[tid] = 0;
    }
    for (int i = tid; i < RANK_BY_PAIRS; i += RANK_THREADS) s_ahead[i] = 0;
    if (tid == 0) { s_higher = 0; s_n = 0; s_low = 0ull; s_high = ~0ull; }
    unsigned bits[RANK_READ];                    // the first calls are on their way while the cuts are ordered
    auto load = [&](int base) {
#pragma unroll
        for (int u = 0; u < RANK_READ; ++u) bits[u] = hx_load_bits(ratio, min(base + u * RANK_THREADS + tid, C - 1));
    };
    load(0);
    __syncthreads();
    {
        const int i = tid & RANK_CUTS, from = (tid / (RANK_CUTS + 1)) * ((RANK_CUTS + 1) / 4);
        const unsigned long long mine = s_cut[i];
        int ahead = 0;
#pragma unroll 8
        for (int k = 0; k < (RANK_CUTS + 1) / 4; ++k) ahead += s_cut[from + k] > mine;
        if (ahead) atomicAdd(&s_place[i], ahead);
    }
    __syncthreads();
    if (tid < RANK_CUTS) {
        if (s_place[tid] == b) s_low = s_cut[tid];
        if (s_place[tid] == b - 1) s_high = s_cut[tid];
    }
    __syncthreads();
    // the bucket: low <= key < high (the first has no upper end, the last no lower one)
    const unsigned long long low = s_low, high = s_high;
    int higher = 0;
    for (int base = 0; base < C;) {
        unsigned now[RANK_READ];
#pragma unroll
        for (int u = 0; u < RANK_READ; ++u) now[u] = bits[u];
        const int at = base;
        base += RANK_READ * RANK_THREADS;
        if (base < C) load(base);
#pragma unroll
        for (int u = 0; u < RANK_READ; ++u) {
            const int c = at + u * RANK_THREADS + tid;
            const unsigned long long key = hx_rank_key64(now[u], c);
            const bool in = c < C;
            higher += in && key >= high;
            if (in && key >= low && key < high) {
                const int slot = atomicAdd(&s_n, 1);
                if (slot < RANK_MEMBERS) s_key[slot] = key;
            }
        }
    }
    if (higher) atomicAdd(&s_higher, higher);
    __syncthreads();
    const int n = s_n;
    higher = s_higher;
    if (__builtin_expect(n <= RANK_BY_PAIRS, 1)) {
        // every wavefront takes a share of the bucket and compares all members with it, RANK_GROUPS in each lane at a time
        const int share = (n + WAVES - 1) / WAVES, end = min((wave + 1) * share, n);
        for (int m0 = 0; m0 < n; m0 += RANK_GROUPS * HX_WAVE) {
            unsigned long long mine[RANK_GROUPS];
            int ahead[RANK_GROUPS];
#pragma unroll
            for (int g = 0; g < RANK_GROUPS; ++g) { mine[g] = s_key[min(m0 + g * HX_WAVE + lane, n - 1)]; ahead[g] = 0; }
#pragma unroll 4
            for (int k = wave * share; k < end; ++k) {
                const unsigned long long key = s_key[k];
#pragma unroll
                for (int g = 0; g < RANK_GROUPS; ++g) ahead[g] += key > mine[g];
            }
#pragma unroll
            for (int g = 0; g < RANK_GROUPS; ++g)
                if (m0 + g * HX_WAVE + lane < n && ahead[g]) atomicAdd(&s_ahead[m0 + g * HX_WAVE + lane], ahead[g]);
        }
        __syncthreads();
        for (int i = tid; i < n; i += RANK_THREADS) rank[0xffffffffu - (unsigned)(s_key[i] & 0xffffffffull)] = higher + s_ahead[i];
        return;
    }
    const bool all = n <= RANK_MEMBERS;                      // the members gathered above are all there are
    int room = RANK_MEMBERS;
    if (all) {
        while (room >> 1 >= n) room >>= 1;
        for (int i = n + tid; i < room; i += RANK_THREADS) s_key[i] = 0ull;
    }
    for (int from = 0; from < (all ? 1 : C); from += RANK_MEMBERS) {
        if (!all) {
            for (int i = tid; i < RANK_MEMBERS; i += RANK_THREADS) {
                const int c = min(from + i, C - 1);
                const unsigned long long key = hx_rank_key64(hx_load_bits(ratio, c), c);
                s_key[i] = from + i < C && key >= low && key < high ? key : 0ull;
            }
        }
        __syncthreads();
        // into decreasing order: bitonic merges
        for (int size = 2; size <= room; size <<= 1)
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int i = tid; i < room >> 1; i += RANK_THREADS) {
                    const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                    const unsigned long long x = s_key[lo], y = s_key[hi];
                    if ((x < y) == ((lo & size) == 0)) { s_key[lo] = y; s_key[hi] = x; }
                }
                __syncthreads();
            }
        if (all)
            for (int i = tid; i < n; i += RANK_THREADS) rank[0xffffffffu - (unsigned)(s_key[i] & 0xffffffffull)] = higher + i;
        else {
            for (int c = tid; c < C; c += RANK_THREADS) {    // a call's places are added up by one thread
                const unsigned long long mine = hx_rank_key64(hx_load_bits(ratio, c), c);
                if (mine < low || mine >= high) continue;
                int ahead = 0;
                for (int step = RANK_MEMBERS; step > 0; step >>= 1) {
                    const int next = min(ahead + step, RANK_MEMBERS);      // (the last key may be looked at more than once)
                    ahead = s_key[next - 1] > mine ? next : ahead;
                }
                rank[c] = (from ? rank[c] : higher) + ahead;
            }
            __syncthreads();
        }
    }
}

// Larger queues: sample sort.  256 evenly spaced calls are sorted and serve as splitters; every call
// finds its bucket among them, takes a slot in it, and is moved next to the other members of its
// bucket; a workgroup per bucket then counts, for every member, the larger keys inside the bucket and
// adds the sizes of all higher buckets.  Keys are unique (they end in the call index), so buckets stay
// balanced however many ratios are equal, and the ranks do not depend on the order the slots were
// taken in.
constexpr int RANK_SPLIT = 256;                  // splitters; buckets 0 .. RANK_SPLIT
constexpr int RANK_BUCKETS = RANK_SPLIT + 1;
constexpr int RANK_CHUNK = 2048;                 // bucket members held in LDS at a time

struct RankScratch {
    unsigned long long *split;                   // [RANK_SPLIT] ascending
    unsigned long long *bkey;                    // [C] keys grouped by bucket
    int *hist;                                   // [RANK_BUCKETS] bucket sizes
};

__global__ __launch_bounds__(RANK_SPLIT) void hx_rank_splitters_kernel(const float *ratio, int C, RankScratch w)
{
    __shared__ unsigned long long s[RANK_SPLIT];
    const int t = threadIdx.x;
    const int c = (int)(((long long)t * C) / RANK_SPLIT);
    s[t] = hx_rank_key64(hx_load_bits(ratio, c), c);
    w.hist[t] = 0;
    if (t == 0) w.hist[RANK_SPLIT] = 0;
    __syncthreads();
    for (int k = 2; k <= RANK_SPLIT; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const int l = t ^ j;
            const unsigned long long x = s[t], y = s[l];
            __syncthreads();
            // ascending bitonic network: the lower index of a pair keeps the smaller key when (t & k) == 0
            const bool keep_small = ((t & k) == 0) == (t < l);
            s[t] = keep_small ? (x < y ? x : y) : (x < y ? y : x);
            __syncthreads();
        }
    }
    w.split[t] = s[t];
}

// bucket of a key: the number of splitters below it
__device__ __forceinline__ int hx_rank_bucket(const unsigned long long *split, unsigned long long key)
{
    int lo = 0, hi = RANK_SPLIT;                  // first splitter that is not below the key
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (split[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// every call takes a slot in its bucket; the slot is parked in rank[c].  The calls of a workgroup first
// count themselves per bucket in LDS, then the workgroup reserves its share of every bucket with one
// global atomic per non-empty bucket (one atomic per call would queue up on 257 addresses).
__global__ __launch_bounds__(1024) void hx_rank_slot_kernel(const float *ratio, int32_t *rank, int C, RankScratch w)
{
    __shared__ unsigned long long s_split[RANK_SPLIT];
    __shared__ int s_cnt[RANK_BUCKETS], s_base[RANK_BUCKETS];
    const int t = threadIdx.x;
    if (t < RANK_SPLIT) s_split[t] = w.split[t];
    if (t < RANK_BUCKETS) s_cnt[t] = 0;
    __syncthreads();
    const int c = blockIdx.x * blockDim.x + t;
    int b = 0, local = 0;
    if (c < C) {
        b = hx_rank_bucket(s_split, hx_rank_key64(hx_load_bits(ratio, c), c));
        local = atomicAdd(&s_cnt[b], 1);
    }
    __syncthreads();
    if (t < RANK_BUCKETS && s_cnt[t] > 0) s_base[t] = atomicAdd(&w.hist[t], s_cnt[t]);
    __syncthreads();
    if (c < C) rank[c] = s_base[b] + local;
}

// exclusive prefix of the bucket sizes, by every workgroup for itself (257 values)
__device__ __forceinline__ void hx_rank_starts(const int *hist, int *s_start)
{
    __shared__ int s_part[4];
    const int t = threadIdx.x;                    // the first 256 threads: bucket t (bucket 256 rides with thread 255)
    const int lane = t & (HX_WAVE - 1), wv = t >> 6;
    const int h = t < RANK_SPLIT ? hist[t] : 0;
    int incl = h;
#pragma unroll
    for (int off = 1; off < HX_WAVE; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    if (t < RANK_SPLIT && lane == HX_WAVE - 1) s_part[wv] = incl;
    __syncthreads();
    if (t < RANK_SPLIT) {
        int base = 0;
        for (int k = 0; k < wv; ++k) base += s_part[k];
        s_start[t] = base + incl - h;
        if (t == RANK_SPLIT - 1) { s_start[RANK_SPLIT] = base + incl; s_start[RANK_BUCKETS] = base + incl + hist[RANK_SPLIT]; }
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void hx_rank_scatter_kernel(const float *ratio, const int32_t *rank, int C, RankScratch w)
{
    __shared__ unsigned long long s_split[RANK_SPLIT];
    __shared__ int s_start[RANK_BUCKETS + 1];
    s_split[threadIdx.x] = w.split[threadIdx.x];
    hx_rank_starts(w.hist, s_start);
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    const unsigned long long key = hx_rank_key64(hx_load_bits(ratio, c), c);
    w.bkey[s_start[hx_rank_bucket(s_split, key)] + rank[c]] = key;
}

// workgroup b: rank of every member of bucket b = keys in higher buckets + larger keys in its own
__global__ __launch_bounds__(1024) void hx_rank_within_kernel(int32_t *rank, int C, RankScratch w)
{
    __shared__ unsigned long long s_key[RANK_CHUNK];
    __shared__ int s_start[RANK_BUCKETS + 1];
    hx_rank_starts(w.hist, s_start);
    const int b = blockIdx.x;
    const int m0 = s_start[b], m1 = s_start[b + 1];
    const int higher = C - m1;
    // members in rounds of one per thread, each compared with the whole bucket, which passes through LDS in chunks
    for (int base = m0; base < m1; base += blockDim.x) {                   // same trip count for all threads
        const int i = base + threadIdx.x;
        const unsigned long long mine = i < m1 ? w.bkey[i] : ~0ull;
        int ahead = 0;
        for (int k0 = m0; k0 < m1; k0 += RANK_CHUNK) {
            const int kn = min(RANK_CHUNK, m1 - k0);
            __syncthreads();
            for (int k = threadIdx.x; k < kn; k += blockDim.x) s_key[k] = w.bkey[k0 + k];
            __syncthreads();
            int k = 0;
            for (; k + 8 <= kn; k += 8) {                  // eight independent reads in flight
                unsigned long long kk[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) kk[u] = s_key[k + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) ahead += kk[u] > mine;
            }
            for (; k < kn; ++k) ahead += s_key[k] > mine;
        }
        if (i < m1) rank[0xffffffffu - (unsigned)(mine & 0xffffffffull)] = higher + ahead;
    }
}

// ---- recomputing greedy -------------------------------------------------------------
//
// One workgroup plans the whole queue: the pool tables, the simulated state and the per-call results live in LDS, there
// is no launch between the picks, and nothing is written to memory before the last.
//
// Every remaining call's cost is recomputed after every pick, but not pair by pair.  A candidate's cost is
// max(done_p + x[class_p][class_d], avail_d) + dec_d; it does not fall when its first operand grows, so
//     m[i]  = min over the prefill instances p of class i of done_p
//     r[k]  = min over i of m[i] + x[i][k]
//     best  = min over d of max(r[class_d], avail_d) + dec_d
// is the minimum over all pairs bit for bit (maxima and minima round nothing, the additions have the same operands).
// Prefill instances of one class and the same rates differ by their queue alone, and the one with the shortest
// finishes first for every call: they are one entry ("kind") of the search.  A pick changes one prefill instance
// (its kind's shortest queue: m of one class) and one decode instance (one column of dec).  The pair itself is
// only found for the call that is picked, by the first wavefront, which also adds it to the state.
//
// What bounds it: a pick is a chain (argmax, pair, commit, candidates of the calls that remain, argmax) of some eight
// LDS round trips and a few hundred dependent instructions; 8 calls or 64 make no difference to it.  So every wavefront
// makes the pick for itself from a copy of the pool in its registers -- handing it on would be another barrier and
// two round trips -- and few wavefronts take part: a call is one lane, or several (G) once the remaining calls leave
// lanes idle.  The decode times of the calls stay in LDS, where they fit; a pick rewrites one column.  Calls that were
// picked leave holes: when half of a stage's calls are gone, the rest is dealt to the lanes anew.
// Whole plans, before (every call whose pair a pick touched searched again, pair by pair, by one of 16 wavefronts) and now:
// 64 calls on 8 + 8 instances 338 -> 85 us, 256 on 64 + 64 2500 -> 465, 256 on 256 + 256 3860 -> 1640, 1024 on 64 + 64
// 20100 -> 6320, 1024 on 256 + 256 30600 -> 16900.  (256 on 64 + 64 with four wavefronts instead of eight: 500.)
// With what a stage does not change in registers (transfers, where a group's arrivals lie) and the divisions of a
// commit by multiplication: 64 on 8 + 8 82 -> 78, 256 on 64 + 64 465 -> 443, 256 on 16 + 16 375 -> 350,
// 256 on 256 + 256 1646 -> 1625; with a nominal batch that is no power of two (48), whose division stays one, 465 -> 458, 376 -> 352 and
// 1644 -> 1633.  (The links of the prefill instances in registers as well: 452 for the second.)
constexpr int GREEDY_THREADS = 8 * HX_WAVE;                  // two wavefronts per SIMD
constexpr int GREEDY_MAX_THREADS = HX_GREEDY_MAX_CALLS;      // a lane per call at least
constexpr int GREEDY_K = HX_GREEDY_MAX_INSTANCES / HX_WAVE;
constexpr int GREEDY_ROWS = 8;                               // groups of entries a lane reads at a time, at most
constexpr int GREEDY_MAX_G = 16;                             // lanes per call at most: a row of lanes (a power of two)

// Unsigned division by a number known beforehand, exact for every 32-bit dividend: T. Granlund, P. Montgomery, "Division by
// invariant integers using multiplication" (1994), section 4.
struct HxDivisor {
    unsigned mul;
    int sh1, sh2;
    HxDivisor() = default;
    explicit HxDivisor(unsigned d)
    {
        int l = 0;
        while (l < 32 && (1ull << l) < d) ++l;
        mul = (unsigned)((((1ull << l) - d) << 32) / d + 1);
        sh1 = l < 1 ? l : 1; sh2 = l > 1 ? l - 1 : 0;
    }
    __host__ __device__ unsigned divide(unsigned n) const
    {
        const unsigned t = (unsigned)(((unsigned long long)mul * n) >> 32);
        return (t + ((n - t) >> sh1)) >> sh2;
    }
};

struct GreedyArgs {
    HxModelF m;
    int C, P, D, T;
    const int32_t *L_in, *L_out, *node, *wf;
    const float *elapsed, *tail, *horizon;
    int n_nodes, n_wf;
    const float *p_flops, *p_hbm, *d_flops, *d_hbm, *bw, *lat;
    const int32_t *p_backlog, *p_type, *d_used, *d_cap, *d_batch, *d_qd, *d_type;
    int tokens_per_seq, max_batch;
    HxDivisor by_tokens;                              // by tokens_per_seq
    float inv_bbar;                                   // 1 / m.bbar where multiplying by it is the division (a power of two), else 0
    int32_t *best_p, *best_d, *rank;
    float *best_cost, *ratio;
    int32_t *backlog_out, *used_out, *batch_out, *qd_out;
    int32_t *status;
};

// decode entries: by class, each class padded to whole groups of four, their number to a whole group per lane
constexpr int GREEDY_ENTRIES = HX_GREEDY_MAX_INSTANCES + 4 * kT + 4 * GREEDY_MAX_G;

// the pool in LDS; its arrays lie at fixed places (their addresses cost no registers)
struct __align__(16) GreedyPool {
    float w[GREEDY_ENTRIES], c1[GREEDY_ENTRIES], c2[GREEDY_ENTRIES], kB[GREEDY_ENTRIES];      // decode entries: hint, per-token terms
    int free[GREEDY_ENTRIES], orig[GREEDY_ENTRIES];                   // free tokens, instance (-1: pad)
    int goff[GREEDY_ENTRIES / 4];                                     // of a group of four: where the arrivals at its class begin
    int used[HX_GREEDY_MAX_INSTANCES], batch[HX_GREEDY_MAX_INSTANCES], qd[HX_GREEDY_MAX_INSTANCES];   // decode instances: simulated state
    int cap[HX_GREEDY_MAX_INSTANCES], pos[HX_GREEDY_MAX_INSTANCES], dty[HX_GREEDY_MAX_INSTANCES];     // capacity, entry, class
    float dF[HX_GREEDY_MAX_INSTANCES], dB[HX_GREEDY_MAX_INSTANCES];   // 1/rates
    float pw[HX_GREEDY_MAX_INSTANCES], pF[HX_GREEDY_MAX_INSTANCES], pB[HX_GREEDY_MAX_INSTANCES];      // prefill instances: wait, 1/rates
    int pty[HX_GREEDY_MAX_INSTANCES], kind[HX_GREEDY_MAX_INSTANCES], backlog[HX_GREEDY_MAX_INSTANCES];
    float kw[HX_GREEDY_MAX_INSTANCES], kF[HX_GREEDY_MAX_INSTANCES], kB2[HX_GREEDY_MAX_INSTANCES];     // kinds, by class: shortest wait, 1/rates
    int kfirst[HX_GREEDY_MAX_INSTANCES];                              // first prefill instance of an instance's kind
    float2 link[kT * kT], link_to[kT * kT];                           // 1/bandwidth, latency: by (from, to) and by (to, from)
    int4 red[2][2][GREEDY_MAX_THREADS / HX_WAVE];                     // a wavefront's most urgent call, picks in turn: key, slot, L, O; cost, ratio, call
    int wcnt[GREEDY_MAX_THREADS / HX_WAVE];
    int seg[kT + 1], kseg[kT + 1], cnt[kT], kcnt[kT];                 // entries and kinds of a class begin here; how many there are
};

// the calls in LDS: host (size) and device (offsets), in 4-byte words
struct GreedyCalls {
    int C4;                                                           // calls, rounded up to a multiple of four
    __host__ __device__ explicit GreedyCalls(int C) : C4((C + 3) & ~3) {}
    __host__ __device__ int rec() const { return 0; }                 // int4 per slot: call, L, O
    __host__ __device__ int in() const { return 4 * C4; }             // float4 per call: elapsed, tail, horizon (-1: index out of range)
    __host__ __device__ int out() const { return 8 * C4; }            // int4 per call: pair, cost, ratio
    __host__ __device__ int rank() const { return 12 * C4; }          // per call, -1 until it is picked
    __host__ __device__ int r() const { return 13 * C4; }             // [kT][C4] earliest arrival per decode class
    __host__ __device__ int dec() const { return (13 + kT) * C4; }    // decode times of the calls, as many as there is room for
};

// lanes per call at most: some four groups of entries for each (more lanes only add reductions)
__host__ __device__ inline int greedy_g_max(int n_groups)
{
    int g_max = 1;
    while (g_max < GREEDY_MAX_G && 4 * g_max < n_groups) g_max <<= 1;
    return g_max;
}

// log2 of the lanes per call for the n calls of a stage, on the lanes the stage before left
__host__ __device__ inline int greedy_lg(int n, int lanes, int g_max)
{
    int lg = 0;
    while ((2 << lg) <= g_max && (n << (lg + 1)) <= lanes) ++lg;
    return lg;
}

// the decode times of a stage's calls fit the words for them
__host__ __device__ inline bool greedy_keeps(int per_lane, int n_waves, int dec_words) { return 4 * per_lane * n_waves * HX_WAVE <= dec_words; }

// dec_words: LDS words behind lay.dec()
// K: instances of either side per lane of a wavefront's copy of the pool; TT: classes, or more
template <int K, int TT, int THREADS>
__global__ __launch_bounds__(THREADS) void hx_plan_greedy_kernel(GreedyArgs a, int dec_words)
{
    extern __shared__ __align__(16) float smem[];
    __shared__ GreedyPool s;
    const GreedyCalls lay(a.C);
    int4 *const s_rec = (int4 *)(smem + lay.rec());
    float4 *const s_in = (float4 *)(smem + lay.in());
    int4 *const s_out = (int4 *)(smem + lay.out());
    int *const s_rank = (int *)(smem + lay.rank());
    float *const s_r = smem + lay.r();
    float *const s_dec = smem + lay.dec();

    const int tid = threadIdx.x, NT = blockDim.x;
    const int lane = tid & (HX_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- what the queue and the pool say, read once
    for (int c = tid; c < a.C; c += NT) {
        s_rec[c] = make_int4(c, a.L_in[c], a.L_out[c], 0);
        const int nd = a.node[c], w = a.wf[c];
        const bool ok = nd >= 0 && nd < a.n_nodes && w >= 0 && w < a.n_wf;
        if (!ok) hx_raise(a.status, HX_ERR_INDEX);
        s_in[c] = make_float4(a.elapsed[c], ok ? a.tail[nd] : 0.0f, ok ? fmaxf(a.horizon[w], 0.0f) : -1.0f, 0.0f);
        s_rank[c] = -1;
    }
    for (int p = tid; p < a.P; p += NT) {
        int t = a.p_type[p];
        if (t < 0 || t >= a.T) { hx_raise(a.status, HX_ERR_INDEX); t = 0; }
        const float invF = 1.0f / a.p_flops[p];
        const int bl = a.p_backlog[p];
        s.pF[p] = invF; s.pB[p] = 1.0f / a.p_hbm[p]; s.pty[p] = t; s.backlog[p] = bl; s.pw[p] = hx_prefill_wait(a.m, bl, invF);
    }
    for (int d = tid; d < a.D; d += NT) {
        int t = a.d_type[d];
        if (t < 0 || t >= a.T) { hx_raise(a.status, HX_ERR_INDEX); t = 0; }
        s.used[d] = a.d_used[d]; s.batch[d] = a.d_batch[d]; s.qd[d] = a.d_qd[d]; s.cap[d] = a.d_cap[d];
        s.dF[d] = 1.0f / a.d_flops[d]; s.dB[d] = 1.0f / a.d_hbm[d]; s.dty[d] = t;
    }
    for (int i = tid; i < kT * kT; i += NT) {
        const bool in = i / kT < a.T && i % kT < a.T;
        const int at = (i / kT) * a.T + i % kT;
        const float2 l = make_float2(in ? 1.0f / a.bw[at] : 0.0f, in && a.lat ? a.lat[at] : 0.0f);
        s.link[i] = l; s.link_to[(i % kT) * kT + i / kT] = l;
    }
    for (int e = tid; e < GREEDY_ENTRIES; e += NT) {                       // pads: no room for anything
        s.w[e] = 0.0f; s.c1[e] = 0.0f; s.c2[e] = 0.0f; s.kB[e] = 0.0f; s.free[e] = -1; s.orig[e] = -1;
        if ((e & 3) == 0) s.goff[e >> 2] = 0;
    }
    if (tid < kT) { s.cnt[tid] = 0; s.kcnt[tid] = 0; }
    __syncthreads();
    // the size of the decode classes; the first prefill instance of every kind
    for (int d = tid; d < a.D; d += NT) atomicAdd(&s.cnt[s.dty[d]], 1);
    for (int p = tid; p < a.P; p += NT) {
        const int t = s.pty[p];
        const float F = s.pF[p], B = s.pB[p];
        int first = p;
#pragma unroll 4
        for (int q = p - 1; q >= 0; --q) first = s.pty[q] == t && s.pF[q] == F && s.pB[q] == B ? q : first;
        s.kfirst[p] = first;
        if (first == p) atomicAdd(&s.kcnt[t], 1);
    }
    __syncthreads();
    if (tid <= kT) {
        int e = 0, q = 0;
        for (int t = 0; t < tid; ++t) { e += (s.cnt[t] + 3) & ~3; q += s.kcnt[t]; }
        s.seg[tid] = e; s.kseg[tid] = q;
    }
    __syncthreads();
    for (int d = tid; d < a.D; d += NT) {
        const int t = s.dty[d];
        int e = s.seg[t];
#pragma unroll 4
        for (int q = 0; q < d; ++q) e += s.dty[q] == t;
        const HxDecF x = hx_decode_terms(a.m, s.used[d], s.batch[d], s.qd[d], s.dF[d], s.dB[d]);
        const long long fr = (long long)s.cap[d] - (long long)s.used[d];
        s.w[e] = x.wait; s.c1[e] = x.c1; s.c2[e] = x.c2; s.kB[e] = x.kB;
        s.free[e] = fr < -1 ? -1 : (fr > 2147483647LL ? 2147483647 : (int)fr);
        s.orig[e] = d; s.pos[d] = e;
        s.goff[e >> 2] = t * lay.C4;
    }
    for (int p = tid; p < a.P; p += NT) {
        const int t = s.pty[p], first = s.kfirst[p];
        int q = s.kseg[t];
#pragma unroll 4
        for (int o = 0; o < first; ++o) q += s.pty[o] == t && s.kfirst[o] == o;
        s.kind[p] = q;
        if (first == p) {
            float w = s.pw[p];
#pragma unroll 4
            for (int o = p + 1; o < a.P; ++o) w = s.kfirst[o] == p ? fminf(w, s.pw[o]) : w;
            s.kw[q] = w; s.kF[q] = s.pF[p]; s.kB2[q] = s.pB[p];
        }
    }
    __syncthreads();
    const int n_groups = __builtin_amdgcn_readfirstlane(s.seg[kT]) >> 2, g_max = greedy_g_max(n_groups);

    // Every wavefront keeps the simulated pool in its registers, an instance of either side per lane (K of each), and makes
    // every pick for itself: the same arithmetic everywhere, nothing to hand on, and one barrier a pick.
    int d_ty[K], d_off[K], d_pos[K], d_cap[K], d_used[K], d_qd[K], d_batch[K], d_free[K];
    float d_F[K], d_B[K], d_w[K], d_c1[K], d_c2[K], d_kB[K];
    int p_ty[K], p_kind[K], p_bl[K];
    float p_w[K], p_F[K], p_B[K], p_kw[K];                // p_kw: the shortest wait of the instance's kind
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const bool hd = j * HX_WAVE + lane < a.D, hp = j * HX_WAVE + lane < a.P;
        const int d = hd ? j * HX_WAVE + lane : 0, p = hp ? j * HX_WAVE + lane : 0;
        const int e = s.pos[d];
        d_ty[j] = s.dty[d]; d_off[j] = s.dty[d] * lay.C4; d_pos[j] = e; d_cap[j] = s.cap[d]; d_used[j] = s.used[d]; d_qd[j] = s.qd[d]; d_batch[j] = s.batch[d];
        d_F[j] = s.dF[d]; d_B[j] = s.dB[d]; d_w[j] = s.w[e]; d_c1[j] = s.c1[e]; d_c2[j] = s.c2[e]; d_kB[j] = s.kB[e];
        d_free[j] = hd ? s.free[e] : -1;
        p_ty[j] = s.pty[p]; p_kind[j] = hp ? s.kind[p] : -1; p_bl[j] = s.backlog[p];
        p_w[j] = hp ? s.pw[p] : INFINITY; p_F[j] = s.pF[p]; p_B[j] = s.pB[p]; p_kw[j] = s.kw[s.kind[p]];
    }

    unsigned several = 0;                                 // classes with more than one kind
    for (int i = 0; i < kT; ++i) several |= s.kseg[i + 1] - s.kseg[i] > 1 ? 1u << i : 0u;
    several = __builtin_amdgcn_readfirstlane(several);
    bool over = false, bad = false;                       // reported once, at the end

    int n = a.C, lanes = NT;
    for (int k = 0; k < a.C;) {
        // ---- a stage: the remaining calls in increasing order, G lanes each
        const int n_before = n;
        n = a.C - k;
        if (k > 0) {
            const int4 mine = s_rec[tid < n_before ? tid : 0];
            const bool stays = tid < n_before && s_rank[mine.x] < 0;
            const unsigned long long b = __builtin_amdgcn_ballot_w64(stays);
            if (lane == 0) s.wcnt[wave] = __popcll(b);
            __syncthreads();
            int at = __popcll(b & ((1ull << lane) - 1ull));
            for (int v = 0; v < wave; ++v) at += s.wcnt[v];
            if (stays) s_rec[at] = mine;
            __syncthreads();
        }
        const int lg = greedy_lg(n, lanes, g_max);
        const int G = 1 << lg, n_lanes = n << lg, n_waves = (n_lanes + HX_WAVE - 1) / HX_WAVE;
        lanes = n_waves * HX_WAVE;                            // a wavefront that sits a stage out loses track of the pool
        const int last = n_waves > 1 ? a.C - n / 2 : a.C;     // the stage's picks end here
        const int per_lane = (n_groups + G - 1) >> lg;
        const bool keep = greedy_keeps(per_lane, n_waves, dec_words);
        const int dec_row = 4 * n_waves * HX_WAVE;
        const int slot = tid >> lg, sub = tid & (G - 1);
        const bool has = slot < n;
        bool alive = has;
        const int at = has ? slot : 0;                        // lanes without a call go along with the first one's and write nothing
        const int4 mine = s_rec[at];
        const int L = mine.y, O = mine.z;
        const float4 in = s_in[mine.x];                       // elapsed, tail, horizon
        const HxCallF cf = hx_call_terms(a.m, L, O);
        float *const my_r = s_r + at;                         // [k * C4]
        float *const my_dec = s_dec + 4 * tid;                // [j * dec_row] four decode times of the lane's j-th group
        const int *const my_goff = s.goff + sub;              // [j << lg] of that group
        const float4 *const my_w = (const float4 *)s.w + sub;
        float m[TT];
        float best = INFINITY;
        unsigned ratio_bits = 0;
        // what a stage does not change and a pick reads: the transfers to the classes of the lane's rows (few classes: in
        // registers), and where the arrivals at the classes of its first groups lie
        float x[TT <= 4 ? TT : 1][TT];
        if constexpr (TT <= 4) {
#pragma unroll
            for (int u = 0; u < TT; ++u) {
                const float2 *l = s.link_to + (((u << lg) + sub) & (kT - 1)) * kT;
#pragma unroll
                for (int i = 0; i < TT; ++i) x[u][i] = hx_transfer(cf, l[i].x, l[i].y);
            }
        }
        constexpr int KEPT = THREADS > GREEDY_THREADS ? 0 : GREEDY_ROWS;      // (as the registers allow)
        int off0[KEPT + 1];
#pragma unroll
        for (int u = 0; u < KEPT; ++u) off0[u] = my_goff[(u < per_lane ? u : 0) << lg];

        // r[k] of the lane's call, its lanes a class each
        auto arrivals = [&]() {
            auto rows = [&](auto n_, int k0) {                // N classes of the lane together (more lanes than classes: some twice)
                constexpr int N = decltype(n_)::value;
                float r[N];
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const float2 *l = s.link_to + ((k0 + (u << lg) + sub) & (kT - 1)) * kT;
                    r[u] = INFINITY;
#pragma unroll
                    for (int i = 0; i < TT; i += 2) {         // a class without instances, or beyond T: +inf
                        if constexpr (TT <= 4) r[u] = fminf(r[u], fminf(m[i] + x[u][i], m[i + 1] + x[u][i + 1]));
                        else {
                            const float4 y = *(const float4 *)(l + i);
                            r[u] = fminf(r[u], fminf(m[i] + hx_transfer(cf, y.x, y.y), m[i + 1] + hx_transfer(cf, y.z, y.w)));
                        }
                    }
                }
                if (alive) {                                  // (a picked call's may be being read)
#pragma unroll
                    for (int u = 0; u < N; ++u) my_r[((k0 + (u << lg) + sub) & (kT - 1)) * lay.C4] = r[u];
                }
            };
            if (a.T <= G) rows(std::integral_constant<int, 1>{}, 0);
            else if (a.T <= 2 * G) rows(std::integral_constant<int, 2>{}, 0);
            else for (int k0 = 0; k0 < a.T; k0 += 4 * G) rows(std::integral_constant<int, 4>{}, k0);
            hx_wave_sync();
        };
        auto decode_time = [&](int fr, float c1, float c2, float kB) {
            return hx_fits(L, O, fr) ? hx_decode_time(cf, c1, c2, kB) : INFINITY;
        };
        auto decode_times = [&](int g) {
            const int4 fr = ((const int4 *)s.free)[g];
            const float4 c1 = ((const float4 *)s.c1)[g], c2 = ((const float4 *)s.c2)[g], kB = ((const float4 *)s.kB)[g];
            return make_float4(decode_time(fr.x, c1.x, c2.x, kB.x), decode_time(fr.y, c1.y, c2.y, kB.y),
                               decode_time(fr.z, c1.z, c2.z, kB.z), decode_time(fr.w, c1.w, c2.w, kB.w));
        };
        // The lowest cost of the lane's call and its ratio, Eq. (2).  N of the lane's groups at a time, read together (past
        // the last the lane's first once more).  Where the arrivals of the first lie is known but for two at a time: such a search
        // has many rows, and asking at each whether it is the first cost more (256 calls on 256 + 256 1645 -> 1670 us).
        auto search_by = [&](auto n_) {
            constexpr int N = decltype(n_)::value;
            float v = INFINITY;
            for (int row = 0; row < per_lane; row += N) {
                float r[N];
                float4 w[N], t[N];
                int off[N];
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const int at_row = row + u < per_lane ? row + u : 0;
                    off[u] = N > 2 && u < KEPT && row == 0 ? off0[u < KEPT ? u : 0] : my_goff[at_row << lg];
                    w[u] = my_w[at_row << lg];
                    t[u] = N > 2 ? *(const float4 *)(my_dec + at_row * dec_row) : decode_times(sub + (at_row << lg));
                }
#pragma unroll
                for (int u = 0; u < N; ++u) r[u] = my_r[off[u]];
#pragma unroll
                for (int u = 0; u < N; ++u)
                    v = fminf(v, fminf(fminf(hx_candidate(r[u], w[u].x, t[u].x), hx_candidate(r[u], w[u].y, t[u].y)),
                                       fminf(hx_candidate(r[u], w[u].z, t[u].z), hx_candidate(r[u], w[u].w, t[u].w))));
            }
            best = hx_lanes_min(v, G);
            ratio_bits = hx_ratio_bits(in.x, best, in.y, in.z, in.z >= 0.0f);
        };
        auto search = [&]() {
            if (!keep) search_by(std::integral_constant<int, 2>{});
            else if (per_lane <= 4) search_by(std::integral_constant<int, 4>{});
            else search_by(std::integral_constant<int, (THREADS > GREEDY_THREADS ? 4 : 8)>{});      // (as the registers allow)
        };

        if (wave < n_waves) {
#pragma unroll
            for (int i = 0; i < TT; ++i) {
                m[i] = INFINITY;
                if (i < a.T)
                    for (int q = s.kseg[i]; q < s.kseg[i + 1]; ++q)
                        m[i] = fminf(m[i], hx_prefill_done(cf, s.kw[q], s.kF[q], s.kB2[q]));
            }
            if (keep) {
                float *q = my_dec;
                for (int j = 0; j < per_lane; ++j, q += dec_row) *(float4 *)q = decode_times(sub + (j << lg));
            }
            arrivals();
            search();
        }

        if (wave >= n_waves) {                                // no calls here any more
            if (n_waves > 1)
                for (int i = k; i < last; ++i) __syncthreads();
            k = last;
        }
        for (; k < last; ++k) {
            // (1) the most urgent remaining call: largest ratio, lowest index among equals (slots, and with them lanes and
            // wavefronts, are in index order)
            const float key = alive ? hx_rank_key(ratio_bits) : -INFINITY;
            const float top = hx_wave_max(key);
            // (no lane with a call: lane 0 stands in; its -inf and "no slot" lose to every wavefront that has one)
            const unsigned long long at_top = __builtin_amdgcn_ballot_w64(alive && key == top);
            int from = at_top ? __builtin_ctzll(at_top) : 0;
            int pick = at_top ? (wave * HX_WAVE + from) >> lg : 0x7fffffff;
            int pL = __builtin_amdgcn_readlane(L, from), pO = __builtin_amdgcn_readlane(O, from);
            float cost = hx_lane_value(best, from);
            int p_ratio = __builtin_amdgcn_readlane((int)ratio_bits, from), call = __builtin_amdgcn_readlane(mine.x, from);
            if (n_waves > 1) {
                if (lane == 0) {
                    s.red[k & 1][0][wave] = make_int4(__float_as_int(top), pick, pL, pO);
                    s.red[k & 1][1][wave] = make_int4(__float_as_int(cost), p_ratio, call, 0);
                }
                __syncthreads();
                const int v = min(lane, n_waves - 1);         // (n_waves is at most a row of lanes; lanes beyond repeat the last)
                const int4 q = s.red[k & 1][0][v], q2 = s.red[k & 1][1][v];
                const float all = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(-hx_lanes_min(-__int_as_float(q.x), n_waves))));
                from = __builtin_ctzll(__builtin_amdgcn_ballot_w64(q.y != 0x7fffffff && __int_as_float(q.x) == all));
                pick = __builtin_amdgcn_readlane(q.y, from);
                pL = __builtin_amdgcn_readlane(q.z, from); pO = __builtin_amdgcn_readlane(q.w, from);
                cost = __int_as_float(__builtin_amdgcn_readlane(q2.x, from)); p_ratio = __builtin_amdgcn_readlane(q2.y, from);
                call = __builtin_amdgcn_readlane(q2.z, from);
            }
            // (2) its pair: for every decode instance that attains the minimum (nearly always one) the lowest prefill
            // instance that does so with it; the lowest (p, d) of these
            int p = -1, d = -1;
            if (cost < INFINITY) {
                const HxCallF pc = hx_call_terms(a.m, pL, pO);
                float done[K], dt[K];
                unsigned long long todo[K];
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    const float r = s_r[d_off[j] + pick];
                    done[j] = hx_prefill_done(pc, p_w[j], p_F[j], p_B[j]);
                    dt[j] = hx_fits(pL, pO, d_free[j]) ? hx_decode_time(pc, d_c1[j], d_c2[j], d_kB[j]) : INFINITY;
                    todo[j] = __builtin_amdgcn_ballot_w64(hx_candidate(r, d_w[j], dt[j]) == cost);
                }
                int best_p = 0x7fffffff;
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    while (todo[j]) {
                        const int ld = __builtin_ctzll(todo[j]);
                        todo[j] &= todo[j] - 1;
                        const float q_w = hx_lane_value(d_w[j], ld), q_dt = hx_lane_value(dt[j], ld);
                        const int q_t = __builtin_amdgcn_readlane(d_ty[j], ld);
                        int low = 0x7fffffff;
#pragma unroll
                        for (int i = K - 1; i >= 0; --i) {
                            const float2 l = s.link[p_ty[i] * kT + q_t];
                            const unsigned long long b = __builtin_amdgcn_ballot_w64(hx_candidate(done[i] + hx_transfer(pc, l.x, l.y), q_w, q_dt) == cost);
                            low = b ? i * HX_WAVE + __builtin_ctzll(b) : low;
                        }
                        if (low < best_p) { best_p = low; d = j * HX_WAVE + ld; }      // decode instances come in order
                    }
                }
                p = best_p != 0x7fffffff ? best_p : -1;
            }
            if (tid == 0) {
                s_rank[call] = k; s_out[call] = make_int4(p, p < 0 ? -1 : d, __float_as_int(cost), p_ratio);
            }
            alive = alive && slot != pick;
            if (p < 0) continue;                              // nothing changes
            // (3) what it adds to the state: every lane works it out for its own instances, the pair's keep it
            const bool valid = pL >= 0 && pO >= 0;
            const int add_L = valid ? pL : 0, add_O = valid ? pO : 0;
            bad = bad || !valid;
            int e = 0, ic = 0, kind = 0, n_free = 0;
            float was = 0.0f, kF = 0.0f, kB = 0.0f, n_c1 = 0.0f, n_c2 = 0.0f, n_kB = 0.0f;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const int n_bl = __builtin_elementwise_add_sat(p_bl[j], add_L);
                const float n_w = hx_prefill_wait(a.m, n_bl, p_F[j]);
                if (K == 1 || (p >> 6) == j) {
                    const int lp = p & (HX_WAVE - 1);
                    ic = __builtin_amdgcn_readlane(p_ty[j], lp); kind = __builtin_amdgcn_readlane(p_kind[j], lp);
                    was = hx_lane_value(p_kw[j], lp); kF = hx_lane_value(p_F[j], lp); kB = hx_lane_value(p_B[j], lp);
                    if (lane == lp) {
                        over = over || n_bl - p_bl[j] != add_L;
                        p_bl[j] = n_bl; p_w[j] = n_w;
                    }
                }
            }
            float now = INFINITY;
#pragma unroll
            for (int j = 0; j < K; ++j) now = p_kind[j] == kind ? fminf(now, p_w[j]) : now;
            now = hx_wave_min(now);
#pragma unroll
            for (int j = 0; j < K; ++j) p_kw[j] = p_kind[j] == kind ? now : p_kw[j];
            if (lane == 0) s.kw[kind] = now;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                if (K == 1 || (d >> 6) == j) {
                    const int n_qd = __builtin_elementwise_add_sat(d_qd[j], add_O);
                    const int us = __builtin_elementwise_add_sat(d_used[j], add_L), n_us = __builtin_elementwise_add_sat(us, add_O);
                    // ceil(us / tokens_per_seq), rounded towards 0: both numbers are below 2^31, so 32 unsigned bits do
                    const int num = n_us < 0 ? n_us + (a.tokens_per_seq - 1) : 0;
                    const unsigned top = n_us < 0 ? (unsigned)(num < 0 ? -num : num) : (unsigned)n_us + (unsigned)a.tokens_per_seq - 1u;
                    const unsigned quot = a.by_tokens.divide(top);
                    const int n_batch = num < 0 ? -(int)quot : (quot > (unsigned)a.max_batch ? a.max_batch : (int)quot);
                    // the derived table entries, by the function that made them
                    const HxDecF x = hx_decode_terms(a.m, n_us, n_batch, n_qd, d_F[j], d_B[j], KEPT ? a.inv_bbar : 0.0f);
                    const int n_fr = max(__builtin_elementwise_sub_sat(d_cap[j], n_us), -1);
                    const int ld = d & (HX_WAVE - 1);
                    if (lane == ld) {
                        over = over || n_qd - d_qd[j] != add_O || us - d_used[j] != add_L || n_us - us != add_O;
                        d_qd[j] = n_qd; d_used[j] = n_us; d_batch[j] = n_batch;
                        d_w[j] = x.wait; d_c1[j] = x.c1; d_c2[j] = x.c2; d_kB[j] = x.kB; d_free[j] = n_fr;
                        s.w[d_pos[j]] = x.wait; s.c1[d_pos[j]] = x.c1; s.c2[d_pos[j]] = x.c2; s.kB[d_pos[j]] = x.kB;
                        s.free[d_pos[j]] = d_free[j];
                    }
                    e = __builtin_amdgcn_readlane(d_pos[j], ld); n_free = __builtin_amdgcn_readlane(d_free[j], ld);
                    n_c1 = hx_lane_value(d_c1[j], ld); n_c2 = hx_lane_value(d_c2[j], ld); n_kB = hx_lane_value(d_kB[j], ld);
                }
            }
            hx_wave_sync();
            // (4) the calls that remain, against the new state
            if (__builtin_amdgcn_ballot_w64(alive) == 0) continue;
            if (keep && sub == ((e >> 2) & (G - 1))) my_dec[(e >> (2 + lg)) * dec_row + (e & 3)] = decode_time(n_free, n_c1, n_c2, n_kB);
            bool moved = now != was;
            if (moved) {
                // the kind's shortest queue has grown (or, with a strange model, shrunk): m of its class grows with it, or
                // falls back to the class's next kind -- if this kind held the minimum
                float v = hx_prefill_done(cf, now, kF, kB);
                if ((several >> ic) & 1) {
                    const float before = hx_prefill_done(cf, was, kF, kB);
                    float mc = m[0];
#pragma unroll
                    for (int i = 1; i < TT; ++i) mc = i == ic ? m[i] : mc;
                    moved = __builtin_amdgcn_ballot_w64(before == mc) != 0 || now < was;
                    if (moved) {
                        const int q_end = s.kseg[ic + 1];
                        for (int q = s.kseg[ic] + sub; q < q_end; q += G) v = fminf(v, hx_prefill_done(cf, s.kw[q], s.kF[q], s.kB2[q]));
                        v = hx_lanes_min(v, G);
                    }
                }
                if (moved) {
#pragma unroll
                    for (int i = 0; i < TT; ++i) m[i] = i == ic ? v : m[i];
                }
            }
            if (moved) arrivals();
            search();
        }
        __syncthreads();
    }
    // ---- the plan, and the simulated state it leaves
    for (int c = tid; c < a.C; c += NT) {
        const int4 q = s_out[c];
        a.best_p[c] = q.x; a.best_d[c] = q.y; a.best_cost[c] = __int_as_float(q.z); a.rank[c] = s_rank[c];
        hx_store_bits(a.ratio, c, (unsigned)q.w);
    }
    if (wave == 0) {
        if (bad) hx_raise(a.status, HX_ERR_INDEX);
        if (over) hx_raise(a.status, HX_ERR_OVERFLOW);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int i = j * HX_WAVE + lane;
            if (i < a.P && a.backlog_out) a.backlog_out[i] = p_bl[j];
            if (i < a.D && a.used_out) a.used_out[i] = d_used[j];
            if (i < a.D && a.batch_out) a.batch_out[i] = d_batch[j];
            if (i < a.D && a.qd_out) a.qd_out[i] = d_qd[j];
        }
    }
}

__global__ __launch_bounds__(256) void hx_plan_no_pool_kernel(GreedyArgs a)
{
    // with an empty pool nothing is feasible: every call has infinite ratio and is ranked by index
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.C) return;
    a.best_p[c] = -1; a.best_d[c] = -1; a.best_cost[c] = INFINITY; a.rank[c] = c;
    hx_projected_ratio(a.node, a.wf, a.elapsed, a.tail, a.horizon, a.n_nodes, a.n_wf, c, INFINITY, a.status, a.ratio);
}

__global__ __launch_bounds__(256) void hx_copy_i32_kernel(const int32_t *src, int32_t *dst, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

}  // namespace

// the planner kernel may use all of a CU's LDS; said once per process
constexpr int GREEDY_LDS = 160 * 1024;
static_assert(sizeof(GreedyPool) + 4 * (13 + kT) * (size_t)HX_GREEDY_MAX_CALLS <= GREEDY_LDS, "the longest queue fits");
int hx_plan_init()
{
    const int most = GREEDY_LDS - (int)sizeof(GreedyPool);
    hipError_t e = hipSuccess;
    auto allow = [&](const void *kernel) {
        if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    };
    allow(reinterpret_cast<const void *>(hx_plan_greedy_kernel<1, 4, GREEDY_THREADS>));
    allow(reinterpret_cast<const void *>(hx_plan_greedy_kernel<1, kT, GREEDY_THREADS>));
    allow(reinterpret_cast<const void *>(hx_plan_greedy_kernel<GREEDY_K, kT, GREEDY_THREADS>));
    allow(reinterpret_cast<const void *>(hx_plan_greedy_kernel<GREEDY_K, kT, GREEDY_MAX_THREADS>));
    return e == hipSuccess ? HX_OK : HX_ERR_DEVICE;
}

extern "C" int hx_rank(hx_ctx *ctx, int32_t C, const float *ratio, int32_t *rank, void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HX_REQUIRE(ctx, C >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, C == 0 || (ratio && rank), HX_ERR_INVALID_ARG, "NULL array");
    if (C == 0) return HX_OK;
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;
    const int bx = (C + 255) / 256;
    if (C <= RANK_DIRECT) {
        hx_rank_direct_kernel<<<(C + HX_WAVE - 1) / HX_WAVE, RANK_THREADS, 0, stream>>>(ratio, rank, C);
        return hx_check_launch(ctx, "hx_rank_direct_kernel");
    }
    if (C <= RANK_PAIRS) {
        // small queues: every call against every call, no scratch.  Tiles short enough for a few thousand
        // workgroups (a workgroup's time is its tile's length, whatever the queue's), long enough to be worth
        // their atomics.
        int tile = (C / 32 + 63) / 64 * 64;
        if (tile < 64) tile = 64;
        if (tile > RANK_TILE) tile = RANK_TILE;
        const int by = (C + tile - 1) / tile;
        hx_rank_zero_kernel<<<bx, 256, 0, stream>>>(rank, C);
        hx_rank_count_kernel<<<dim3(bx, by), 256, 0, stream>>>(ratio, rank, C, tile);
        return hx_check_launch(ctx, "hx_rank kernels");
    }
    if (C <= RANK_CUT) {
        hx_rank_cut_kernel<<<RANK_CUTS + 1, RANK_THREADS, 0, stream>>>(ratio, rank, C);
        return hx_check_launch(ctx, "hx_rank_cut_kernel");
    }
    const size_t need = (size_t)C + RANK_SPLIT + (RANK_BUCKETS + 1) / 2 + 8;      // keys, splitters, bucket sizes (two ints per word)
    if (need > ctx->rkey_cap) {
        // grown, never shrunk; work queued on the old block has to finish before it goes
        HX_HIP(ctx, hipDeviceSynchronize());
        if (ctx->d_rkey) { HX_HIP(ctx, hipFree(ctx->d_rkey)); ctx->d_rkey = nullptr; ctx->rkey_cap = 0; }
        HX_HIP(ctx, hipMalloc((void **)&ctx->d_rkey, need * sizeof(unsigned long long)));
        ctx->rkey_cap = need;
    }
    RankScratch w;
    w.split = ctx->d_rkey;
    w.bkey = ctx->d_rkey + RANK_SPLIT;
    w.hist = (int *)(ctx->d_rkey + RANK_SPLIT + C);
    hx_rank_splitters_kernel<<<1, RANK_SPLIT, 0, stream>>>(ratio, C, w);
    hx_rank_slot_kernel<<<(C + 1023) / 1024, 1024, 0, stream>>>(ratio, rank, C, w);
    hx_rank_scatter_kernel<<<bx, 256, 0, stream>>>(ratio, rank, C, w);
    hx_rank_within_kernel<<<RANK_BUCKETS, 1024, 0, stream>>>(rank, C, w);
    return hx_check_launch(ctx, "hx_rank kernels");
}

struct GreedyLaunch {
    int threads;
    size_t lds;
    int dec_words;
};

static GreedyLaunch greedy_launch(int C, int D, int T)
{
    // A lane per call where the pool is small (a wavefront that is alone has no barriers); otherwise a lane for every
    // four groups of decode entries, as long as that leaves two wavefronts per SIMD (a lane for every two: 472 us
    // instead of 465 for 256 calls on 64 + 64, and no difference for 64 on 8 + 8).
    const int groups = (D + 3) / 4;
    int threads = C;
    while (threads < GREEDY_THREADS && threads < C * ((groups + 3) / 4)) threads *= 2;
    threads = (threads + HX_WAVE - 1) / HX_WAVE * HX_WAVE;
    if (threads < HX_WAVE) threads = HX_WAVE;
    if (threads > GREEDY_THREADS && C <= GREEDY_THREADS) threads = GREEDY_THREADS;
    const GreedyCalls lay(C);
    // room for the decode times of every call, as far as the LDS goes (what does not fit is worked out at each pick)
    const size_t room = GREEDY_LDS - sizeof(GreedyPool) - 4 * lay.dec();
    size_t lds = (size_t)threads * 16 * (((size_t)groups + T) * C / threads + 2);
    lds = 4 * lay.dec() + (lds < room ? lds : room);
    return {threads, lds, (int)(lds / 4) - lay.dec()};
}

// for tests: of a plan's stages, with n_groups groups of four decode entries, is there one whose decode times are kept (1), one
// whose are not (2), both (3)
extern "C" int hx_test_plan_stages(int C, int D, int T, int n_groups)
{
    if (C < 1 || C > HX_GREEDY_MAX_CALLS || D < 1 || D > HX_GREEDY_MAX_INSTANCES || T < 1 || T > HX_MAX_TYPES) return HX_ERR_SHAPE;
    const GreedyLaunch g = greedy_launch(C, D, T);
    int seen = 0;
    for (int n = C, lanes = g.threads; n > 0;) {
        const int lg = greedy_lg(n, lanes, greedy_g_max(n_groups)), n_waves = ((n << lg) + HX_WAVE - 1) / HX_WAVE;
        seen |= greedy_keeps((n_groups + (1 << lg) - 1) >> lg, n_waves, g.dec_words) ? 1 : 2;
        lanes = n_waves * HX_WAVE;
        n = n_waves > 1 ? n / 2 : 0;
    }
    return seen;
}

extern "C" int hx_plan_greedy(hx_ctx *ctx, const hx_model *model, const hx_calls *calls,
                              const hx_prefill_tab *pre, const hx_decode_tab *dec, const hx_links *links,
                              const float *tail, const float *horizon, int32_t n_nodes, int32_t n_wf,
                              int32_t tokens_per_seq, int32_t max_batch,
                              int32_t *best_p, int32_t *best_d, float *best_cost, float *ratio, int32_t *rank,
                              int32_t *backlog_tok_out, int32_t *used_tok_out, int32_t *batch_out, int32_t *qd_tok_out,
                              void *stream_)
{
    if (!ctx) return HX_ERR_INVALID_ARG;
    HX_REQUIRE(ctx, model && calls && pre && dec && links, HX_ERR_INVALID_ARG, "NULL table");
    const int C = calls->n, P = pre->n, D = dec->n, T = links->n_types;
    HX_REQUIRE(ctx, C >= 0, HX_ERR_INVALID_ARG, "negative size");
    HX_REQUIRE(ctx, C <= HX_GREEDY_MAX_CALLS, HX_ERR_SHAPE, "%d calls beyond the %d the recomputing planner takes", C,
               HX_GREEDY_MAX_CALLS);
    HX_REQUIRE(ctx, P <= HX_GREEDY_MAX_INSTANCES && D <= HX_GREEDY_MAX_INSTANCES, HX_ERR_SHAPE,
               "pool %d x %d beyond the %d instances per side the recomputing planner takes", P, D, HX_GREEDY_MAX_INSTANCES);
    HX_REQUIRE(ctx, tokens_per_seq > 0 && max_batch >= 0, HX_ERR_INVALID_ARG, "tokens_per_seq must be positive");
    HX_REQUIRE(ctx, best_p && best_d && best_cost && ratio && rank, HX_ERR_INVALID_ARG, "NULL output");
    HX_REQUIRE(ctx, C == 0 || (calls->L_in && calls->L_out && calls->node && calls->wf && calls->elapsed && tail && horizon),
               HX_ERR_INVALID_ARG, "the planner needs L_in, L_out, node, wf, elapsed, tail and horizon");
    HX_REQUIRE(ctx, n_nodes >= 0 && n_wf >= 0, HX_ERR_INVALID_ARG, "negative n_nodes or n_wf");
    HxDeviceGuard guard(ctx->device);
    HX_REQUIRE(ctx, guard.ok, HX_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipStream_t stream = (hipStream_t)stream_;

    GreedyArgs a{};
    a.m = HxModelF{model->kv_bytes_per_token, model->flops_per_token, model->attn_flops_per_token2,
                   model->weight_bytes, model->nominal_batch};
    a.C = C; a.P = P; a.D = D;
    a.L_in = calls->L_in; a.L_out = calls->L_out; a.node = calls->node; a.wf = calls->wf; a.elapsed = calls->elapsed;
    a.tail = tail; a.horizon = horizon; a.n_nodes = n_nodes; a.n_wf = n_wf;
    a.T = links->n_types; a.bw = links->bw; a.lat = links->latency;
    a.p_flops = pre->flops; a.p_hbm = pre->hbm_bw; a.p_backlog = pre->backlog_tok; a.p_type = pre->type;
    a.d_flops = dec->flops; a.d_hbm = dec->hbm_bw; a.d_used = dec->used_tok; a.d_cap = dec->cap_tok;
    a.d_batch = dec->batch; a.d_qd = dec->qd_tok; a.d_type = dec->type;
    a.tokens_per_seq = tokens_per_seq; a.max_batch = max_batch; a.by_tokens = HxDivisor((unsigned)tokens_per_seq);
    int exponent = 0;
    a.inv_bbar = std::frexp(a.m.bbar, &exponent) == 0.5f && std::abs(exponent) < 64 ? 1.0f / a.m.bbar : 0.0f;
    a.best_p = best_p; a.best_d = best_d; a.rank = rank; a.best_cost = best_cost; a.ratio = ratio;
    a.backlog_out = backlog_tok_out; a.used_out = used_tok_out; a.batch_out = batch_out; a.qd_out = qd_tok_out;
    a.status = ctx->d_status;

    if (P == 0 || D == 0) {
        // an empty side: nothing is feasible, the state is returned unchanged
        if (P) HX_REQUIRE(ctx, pre->backlog_tok, HX_ERR_INVALID_ARG, "NULL member in prefill table");
        if (D) HX_REQUIRE(ctx, dec->used_tok && dec->batch && dec->qd_tok, HX_ERR_INVALID_ARG, "NULL member in decode table");
        if (C) hx_plan_no_pool_kernel<<<(C + 255) / 256, 256, 0, stream>>>(a);
        if (P && backlog_tok_out) hx_copy_i32_kernel<<<(P + 255) / 256, 256, 0, stream>>>(pre->backlog_tok, backlog_tok_out, P);
        if (D && used_tok_out) hx_copy_i32_kernel<<<(D + 255) / 256, 256, 0, stream>>>(dec->used_tok, used_tok_out, D);
        if (D && batch_out) hx_copy_i32_kernel<<<(D + 255) / 256, 256, 0, stream>>>(dec->batch, batch_out, D);
        if (D && qd_tok_out) hx_copy_i32_kernel<<<(D + 255) / 256, 256, 0, stream>>>(dec->qd_tok, qd_tok_out, D);
        return hx_check_launch(ctx, "hx_plan_no_pool_kernel");
    }
    if (int rc = hx_check_pool(ctx, model, pre, dec, links)) return rc;
    const GreedyLaunch g = greedy_launch(C, D, T);
    auto launch = [&](auto kernel) { kernel<<<1, g.threads, g.lds, stream>>>(a, g.dec_words); };
    if (g.threads > GREEDY_THREADS) launch(hx_plan_greedy_kernel<GREEDY_K, kT, GREEDY_MAX_THREADS>);
    else if (P > HX_WAVE || D > HX_WAVE) launch(hx_plan_greedy_kernel<GREEDY_K, kT, GREEDY_THREADS>);
    else if (T > 4) launch(hx_plan_greedy_kernel<1, kT, GREEDY_THREADS>);
    else launch(hx_plan_greedy_kernel<1, 4, GREEDY_THREADS>);
    return hx_check_launch(ctx, "hx_plan_greedy_kernel");
}
