// What the scoring kernels, the planners and the decode stage share: reductions over a wavefront and the
// projected ratio, so that all of them round and order alike.
#pragma once

#include "hx_common.hpp"
#include "hx_terms.hpp"

#include <cmath>

// Minimum over the 64 lanes of a wavefront with data-parallel-primitive lane
// moves (no LDS traffic): two quad swaps and two row mirrors leave every row
// of 16 lanes holding its minimum, two row broadcasts carry it to lane 63,
// which is read back as a wave-uniform value.  Each step is one instruction,
// the minimum itself taking its first operand through the lane move (lanes
// a row mask leaves out keep their value: the destination is the operand).
// A lane move may read a register two cycles after a vector instruction wrote
// it at the earliest, and five after one wrote the execution mask; the
// compiler does not see inside these statements, so they carry their own waits
// (and one at the end, before the lane read that follows).
#define HX_DPP_MIN_CHAIN(OP)                                                                  \
    "s_nop 4\n\t" OP " %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"        \
    "s_nop 1\n\t" OP " %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"        \
    "s_nop 1\n\t" OP " %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"            \
    "s_nop 1\n\t" OP " %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"                 \
    "s_nop 1\n\t" OP " %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"               \
    "s_nop 1\n\t" OP " %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"               \
    "s_nop 1"

__device__ __forceinline__ float hx_wave_min(float x)
{
    asm volatile(HX_DPP_MIN_CHAIN("v_min_f32_dpp") : "+v"(x));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

__device__ __forceinline__ int hx_wave_min(int x)
{
    asm volatile(HX_DPP_MIN_CHAIN("v_min_i32_dpp") : "+v"(x));
    return __builtin_amdgcn_readlane(x, 63);
}

__device__ __forceinline__ float hx_wave_max(float x)
{
    asm volatile(HX_DPP_MIN_CHAIN("v_max_f32_dpp") : "+v"(x));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// The wavefront's largest value and the lowest index that has it, in every lane.  A lane without a
// candidate passes (-inf, INT_MAX): it loses to every candidate, also to one whose value is -inf.
// Every lane of the wavefront must be active.
__device__ __forceinline__ void hx_wave_argmax(float &v, int &i)
{
    const float top = hx_wave_max(v);
    i = hx_wave_min(v == top ? i : 0x7fffffff);
    v = top;
}

// The minimum over the groups of G neighbouring lanes (G a power of two, at most a row of 16; other G: the next one), in each lane.
__device__ __forceinline__ float hx_lanes_min(float x, int G)
{
#define HX_ROW_MIN(ctrl) x = fminf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), ctrl, 0xf, 0xf, true)))
    if (G > 1) HX_ROW_MIN(0xB1);           // quad_perm [1,0,3,2]
    if (G > 2) HX_ROW_MIN(0x4E);           // quad_perm [2,3,0,1]
    if (G > 4) HX_ROW_MIN(0x141);          // row_half_mirror
    if (G > 8) HX_ROW_MIN(0x140);          // row_mirror
#undef HX_ROW_MIN
    return x;
}

__device__ __forceinline__ int hx_lanes_min(int x, int G)
{
#define HX_ROW_MIN(ctrl) x = min(x, __builtin_amdgcn_mov_dpp(x, ctrl, 0xf, 0xf, true))
    if (G > 1) HX_ROW_MIN(0xB1);
    if (G > 2) HX_ROW_MIN(0x4E);
    if (G > 4) HX_ROW_MIN(0x141);
    if (G > 8) HX_ROW_MIN(0x140);
#undef HX_ROW_MIN
    return x;
}

// sum over the wavefront; all lanes take part, all have the result
__device__ __forceinline__ unsigned hx_wave_sum(unsigned x)
{
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);      // row_shr 1, 2, 4, 8
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);      // row_bcast 15, 31
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);
    return (unsigned)__builtin_amdgcn_readlane((int)x, HX_WAVE - 1);
}

// of values below 2^31, in 64 bits: by halves, 64 of which fit 32 bits
__device__ __forceinline__ unsigned long long hx_wave_sum_i31(int x)
{
    return (unsigned long long)hx_wave_sum((unsigned)x & 0xffffu) + ((unsigned long long)hx_wave_sum((unsigned)x >> 16) << 16);
}

// LDS written by some lanes of a wavefront and read by others of it
__device__ __forceinline__ void hx_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float hx_lane_value(float x, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane)); }

// The library is built on the assumption that no arithmetic ever sees a NaN, so
// the NaN that marks a bad index is chosen among integers and stored as bits.
constexpr unsigned HX_QNAN_BITS = 0x7fc00000u;

// Eq. (2) with the downstream tail of the call's node, as bits: (elapsed + best
// + tail) / horizon; a workflow without a horizon (0: nothing it has revealed
// costs anything) makes its calls as urgent as can be, +inf; !ok gives the NaN.
__device__ __forceinline__ unsigned hx_ratio_bits(float elapsed, float best, float tail, float horizon, bool ok)
{
    const float r = horizon > 0.0f ? ((elapsed + best) + tail) / horizon : INFINITY;
    return ok ? __float_as_uint(r) : HX_QNAN_BITS;
}

__device__ __forceinline__ void hx_store_bits(float *out, int i, unsigned bits) { ((unsigned *)out)[i] = bits; }

// projected ratio of call c, stored to ratio[c].  A node or workflow index
// outside the arrays gives NaN and raises HX_ERR_INDEX.
__device__ __forceinline__ void hx_projected_ratio(const int32_t *node, const int32_t *wf, const float *elapsed,
                                                   const float *tail, const float *horizon, int n_nodes, int n_wf,
                                                   int c, float best, int32_t *status, float *ratio)
{
    const int nd = node[c], w = wf[c];
    const bool ok = nd >= 0 && nd < n_nodes && w >= 0 && w < n_wf;
    if (!ok) hx_raise(status, HX_ERR_INDEX);
    hx_store_bits(ratio, c, hx_ratio_bits(elapsed[c], best, ok ? tail[nd] : 0.0f, ok ? horizon[w] : 1.0f, ok));
}

// a ratio as it is stored: it may be the NaN, and a float that may be one is not so much as handed to a function
__device__ __forceinline__ unsigned hx_load_bits(const float *in, int i) { return ((const unsigned *)in)[i]; }

// ordering key of a ratio's bits: the NaN (raised elsewhere as a bad index) sorts with +inf
__device__ __forceinline__ float hx_rank_key(unsigned b)
{
    return __uint_as_float((b & 0x7fffffffu) > 0x7f800000u ? 0x7f800000u : b);
}
