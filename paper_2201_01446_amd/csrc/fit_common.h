// fit_common.h -- MFMA fragments, precision conversions and the epilogue
// tanh shared by the fitting-net GEMM (gemm.hip), the fused fitting tail
// (fit.hip) and the compressed step's net (fitnet.hip, fitsplit.hip), and the
// rows, the scheduling and the lane sums of the last two.
#pragma once

#include "dp_internal.h"
#include "tanh64.h"

#include <type_traits>

namespace dp {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef double d2v __attribute__((ext_vector_type(2)));
// 16 raw bytes as a native vector (HIP's uint4 struct defeats register promotion)
typedef unsigned int u4v __attribute__((ext_vector_type(4)));

namespace {

template <typename TA> struct MMT;
template <> struct MMT<double> { using acc = double; using accv = d4v; static constexpr int VEC = 2; };
template <> struct MMT<float> { using acc = float; using accv = f4v; static constexpr int VEC = 4; };
template <> struct MMT<__bf16> { using acc = float; using accv = f4v; static constexpr int VEC = 8; };

// One K-group (4 lanes-groups x VEC elements) of MFMA on 16-byte fragments.
// For the 4-deep FP32/FP64 instructions the VEC elements of a fragment feed
// VEC instructions; lane group q then holds k = q*VEC + v of the group in the
// v-th one, the same mapping for A and B, so the group's sum is complete.
__device__ inline void mfma_frag(const u4v &a, const u4v &b, d4v &c)
{
    d2v x = __builtin_bit_cast(d2v, a), y = __builtin_bit_cast(d2v, b);
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(x[0], y[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(x[1], y[1], c, 0, 0, 0);
}
__device__ inline void mfma_frag_f32(const u4v &a, const u4v &b, f4v &c)
{
    f4v x = __builtin_bit_cast(f4v, a), y = __builtin_bit_cast(f4v, b);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0], y[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[1], y[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[2], y[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[3], y[3], c, 0, 0, 0);
}
__device__ inline void mfma_frag_bf16(const u4v &a, const u4v &b, f4v &c)
{
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a), __builtin_bit_cast(bf8v, b),
                                                c, 0, 0, 0);
}

template <typename TA, typename AV>
__device__ inline void mfma_any(const u4v &a, const u4v &b, AV &c)
{
    if constexpr (std::is_same<TA, double>::value) mfma_frag(a, b, c);
    else if constexpr (std::is_same<TA, float>::value) mfma_frag_f32(a, b, c);
    else mfma_frag_bf16(a, b, c);
}

template <typename T> __device__ inline T to(float v);
template <> __device__ inline float to<float>(float v) { return v; }
template <> __device__ inline double to<double>(float v) { return v; }
template <> __device__ inline __bf16 to<__bf16>(float v) { return (__bf16)v; }
template <typename T> __device__ inline T tod(double v);
template <> __device__ inline float tod<float>(double v) { return (float)v; }
template <> __device__ inline double tod<double>(double v) { return v; }
template <> __device__ inline __bf16 tod<__bf16>(double v) { return (__bf16)(float)v; }

__device__ inline float tanh_r(float v) { return tanhf(v); }
__device__ inline double tanh_r(double v) { return tanh_f64(v); }

// tanh of an epilogue: native, or from the second-order table on [0, 8)
// (odd extension, 1 beyond 8), read in the epilogue's precision.
__device__ inline float tanh_e(float x, const float *tab)
{
    if (!tab) return tanhf(x);
    float ax = fabsf(x);
    if (ax >= 8.f) return copysignf(1.f, x);
    int k = (int)(ax * (kTanhN / 8.f));
    k = k < kTanhN - 1 ? k : kTanhN - 1;
    float t = ax - k * (8.f / kTanhN);
    float4 a = *reinterpret_cast<const float4 *>(tab + 4 * k);
    float y = fmaf(t, fmaf(t, a.z, a.y), a.x);
    return copysignf(y, x);
}
__device__ inline double tanh_e(double x, const double *tab)
{
    if (!tab) return tanh_f64(x);
    double ax = fabs(x);
    if (ax >= 8.0) return copysign(1.0, x);
    int k = (int)(ax * (kTanhN / 8.0));
    k = k < kTanhN - 1 ? k : kTanhN - 1;
    double t = ax - k * (8.0 / kTanhN);
    const double *a = tab + 4 * k;
    double y = fma(t, fma(t, a[2], a[1]), a[0]);
    return copysign(y, x);
}
// The table an epilogue of result type TR takes (NULL: native tanh).
__device__ inline const float *tanh_table_for(const Epi &e, float) { return e.tanh_tab; }
__device__ inline const double *tanh_table_for(const Epi &e, double) { return e.tanh_tab64; }


// ------------------------------------ the compressed step's net (fitnet.hip, fitsplit.hip)
// Rows of the net: row -> atom (-1: padding), and the type group of a tile.
__device__ inline int row_atom(const FitRows &fr, int row)
{
    if (fr.ratom) return fr.ratom[row];
    return row < fr.nlive ? row : -1;
}
__device__ inline int row_type(const FitRows &fr, int row)
{
    int ty = 0;
    for (int g = 1; g < fr.ntr; g++) ty += row >= fr.trow[g] ? 1 : 0;
    return ty;
}

// The wave's number in its block, in a scalar register: what follows from it
// (the weights' addresses) is then computed by the scalar unit.  FP64 MFMA and
// the vector ALU share their pipe, so vector address arithmetic costs MFMA time.
__device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Keeps the loads issued before it where they are: the compiler otherwise
// moves a ring's loads down to their use, a whole turn of the ring later.
__device__ inline void keep_order() { __builtin_amdgcn_sched_barrier(0); }

// UP false: even rows of 16 lanes get a + a of the odd row beside, odd rows
// b + b of the even row; UP true: the same between the halves of 32 lanes.
template <bool UP>
__device__ inline float swap_add(float a, float b)
{
    const unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    auto s = UP ? __builtin_amdgcn_permlane32_swap(x, y, false, false) : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    return __builtin_bit_cast(float, (unsigned)s[0]) + __builtin_bit_cast(float, (unsigned)s[1]);
}
template <bool UP>
__device__ inline double swap_add(double a, double b)
{
    const int2 x = __builtin_bit_cast(int2, a), y = __builtin_bit_cast(int2, b);
    auto s = UP ? __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false) : __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
    auto t = UP ? __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false) : __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    return __builtin_bit_cast(double, int2{(int)s[0], (int)t[0]}) + __builtin_bit_cast(double, int2{(int)s[1], (int)t[1]});
}

// Rows of 16 that a launch covers.
inline int row_tiles(const FitRows &fr) { return fr.ntr > 1 ? fr.trow[fr.ntr] / 16 : div_up(fr.nlive, 16); }

}  // namespace

}  // namespace dp
