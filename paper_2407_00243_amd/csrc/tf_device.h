// Device helpers shared by the kernel sources.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

#include "tf_internal.h"

namespace tf {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <typename T> struct Tr;
// D(16x16) += A(16x4) * B(4x16), one wave.  Lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16].  Afterwards lane l = 16 g + r holds, in component v, D[4 g + v][r] for
// fp32 but D[4 v + g][r] for fp64 (measured on gfx950).  `col_of_m` maps the M index that a
// lane feeds to the column of the C slice it stands for, chosen so that in both precisions
// lane (g, r) ends up with the four consecutive columns 4 g .. 4 g + 3 of row r.
template <> struct Tr<float> {
    static constexpr int V = 4;
    typedef floatx4 Acc;
    __device__ static __forceinline__ int col_of_m(int m) { return m; }
};
template <> struct Tr<double> {
    static constexpr int V = 2;
    typedef doublex4 Acc;
    __device__ static __forceinline__ int col_of_m(int m) { return 4 * (m & 3) + (m >> 2); }
};

__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ doublex4 mfma16(double a, double b, doublex4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <typename T, int N> struct alignas(sizeof(T) * N) Pack {
    T x[N];
};

template <typename T, int N> __device__ __forceinline__ void load_pack(T (&dst)[N], const T *p) {
    const Pack<T, N> v = *reinterpret_cast<const Pack<T, N> *>(p);
#pragma unroll
    for (int i = 0; i < N; ++i) dst[i] = v.x[i];
}
template <typename T, int N> __device__ __forceinline__ void store_pack(T *p, const T (&src)[N]) {
    Pack<T, N> v;
#pragma unroll
    for (int i = 0; i < N; ++i) v.x[i] = src[i];
    *reinterpret_cast<Pack<T, N> *>(p) = v;
}

// Sixteen bytes at any element-aligned address.
template <typename T> struct Piece16;
template <> struct Piece16<float> {
    typedef float Vec __attribute__((ext_vector_type(4), aligned(4)));
};
template <> struct Piece16<double> {
    typedef double Vec __attribute__((ext_vector_type(2), aligned(8)));
};
// The same for device memory: one 16-byte access (N = elements per 16 bytes) or one element (N = 1) at
// any element-aligned address.
template <typename T, int N> __device__ __forceinline__ void load_any(T (&dst)[N], const T *p) {
    static_assert(N == 1 || N == Tr<T>::V, "one element or sixteen bytes");
    if constexpr (N == 1) {
        dst[0] = *p;
    } else {
        const typename Piece16<T>::Vec v = *reinterpret_cast<const typename Piece16<T>::Vec *>(p);
#pragma unroll
        for (int i = 0; i < N; ++i) dst[i] = v[i];
    }
}
template <typename T, int N> __device__ __forceinline__ void store_any(T *p, const T (&src)[N]) {
    static_assert(N == 1 || N == Tr<T>::V, "one element or sixteen bytes");
    if constexpr (N == 1) {
        *p = src[0];
    } else {
        typename Piece16<T>::Vec v;
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = src[i];
        *reinterpret_cast<typename Piece16<T>::Vec *>(p) = v;
    }
}

// fp32 products on the bf16 matrix cores (16 times the rate of the fp32 ones, and unlike these they run beside other vector
// instructions of their SIMD).  x = h + m + l, each rounded to nearest even: 24 bits in three times eight, nothing is lost.
// All products of two parts are exact.  An instruction adds up the eight products that a lane supplies, and the accumulator if it
// is the smaller one, cut off at 2^-24 of the largest (measured), and rounds their sum with the accumulator.  So the products h h,
// of 16 bits, have accumulators of their own, in which little is cut off and one rounding in eight products is made, and
// the small products others, whose errors are below 2^-31; both sums are joined by one rounded addition (split_sum).  With
// both in one accumulator the small ones, or h h of the next step, were cut off: relative error of 40000 x 64 sums of 2 / 8 /
// 16 / 64 products against 64 bits 4.4e-8 / 9.1e-8 / 1.2e-7 / 1.5e-7, by the fp32 instructions 3.1e-8 / 5.3e-8 / 7.4e-8 / 1.5e-7.
// Of the nine products of parts only l l is left out, below 2^-33 of the product; m l and l m come to just under 2^-24 of it
// (0x1.00ff8p0 squared), as much as its rounding (without them single products erred by up to twice that; 2D stencil 512^2, 64 ->
// 64, 30.4 us, so 32.8, R-MAT graph of 2^20 rows, 128 -> 128, 930 us, so 958).
typedef __bf16 Bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 Bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t Word4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, Bf16x2{(__bf16)a, (__bf16)b});
}
// The bf16 matrix cores take numbers below 2^-126 for zeros.  Both operands are therefore multiplied by 2^24 first: the last bit
// of the smallest fp32 number becomes 2^-125, so that no part of any number is lost, and what is lost of a product lies
// below 2^-174 of the result, far under the spacing of the smallest numbers.  Sums come out 2^48 times too large.
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;
// 2^24 a, 2^24 b -> words `at` of the three parts
__device__ __forceinline__ void split_pair(Word4 (&part)[3], int at, float a, float b) {
    a *= kSplitScale;
    b *= kSplitScale;
    const uint32_t h = bf16_pair(a, b);
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    const uint32_t m = bf16_pair(a, b);
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xffff0000u);
    part[0][at] = h;
    part[1][at] = m;
    part[2][at] = bf16_pair(a, b);
}
// D(16x16) += A(16x32) B(32x16), one wave: lane l supplies A[l % 16][8 (l / 16) + q] and B[8 (l / 16) + q][l % 16], q < 8;
// results as for fp32 above.
__device__ __forceinline__ floatx4 mfma16_bf16(const Word4 &a, const Word4 &b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(Bf16x8, a), __builtin_bit_cast(Bf16x8, b), c, 0, 0, 0);
}
// Results from the sums of h h and those of the small products.
__device__ __forceinline__ floatx4 split_sum(const floatx4 &high, const floatx4 &small) {
    floatx4 y;
#pragma unroll
    for (int v = 0; v < 4; ++v) y[v] = (high[v] + small[v]) * kSplitUnscale;
    return y;
}
// A row of the first operand and a column of the second are multiplied this way if their largest elements are below 2^60 and
// the product of these is below 2^72: no sum of 128 products reaches 2^128 then, scaled by 2^48.  Infinities, which would meet
// zeros of the other operand's parts, are beyond as well.
constexpr float kSplitMax = 0x1p60f, kSplitProduct = 0x1p72f;
__device__ __forceinline__ bool split_exceeds(float largest, float bound) { return !(largest < bound); }
// From the largest elements of the columns (bits; a NaN counts as more than infinity): whether one is beyond, and what those
// of a row must be below.
__device__ __forceinline__ float split_row_bound(const uint32_t *cmax, int cols, int lane, bool &exceeds) {
    float most = 0.0f;
    bool any = false;
    for (int c = lane; c < cols; c += 64) {
        const float m = __uint_as_float(cmax[c]);
        any |= split_exceeds(m, kSplitMax);
        most = fmaxf(most, m);
    }
    exceeds = __builtin_amdgcn_ballot_w64(any) != 0;
    // (the exchange of the most takes 0.2 us, which small launches show)
    constexpr float usual = kSplitProduct / kSplitMax;
    if (__builtin_amdgcn_ballot_w64(most > usual) == 0) return kSplitMax;
    for (int i = 1; i < 64; i <<= 1) most = fmaxf(most, __shfl_xor(most, i, 64));
    return kSplitProduct / most;
}
// Eight numbers of an operand in LDS: put together again from their parts, which takes nothing from them, or as they are
// (`whole`) in the place of the first two parts.
__device__ __forceinline__ void split_whole(float (&x)[8], const Word4 *at, bool whole) {
    const Word4 h = at[0], m = at[64];
    if (whole) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            x[q] = __uint_as_float(h[q]);
            x[4 + q] = __uint_as_float(m[q]);
        }
        return;
    }
    const Word4 l = at[128];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        x[2 * q] = (__uint_as_float(h[q] << 16) + (__uint_as_float(m[q] << 16) + __uint_as_float(l[q] << 16))) * (1.0f / kSplitScale);
        x[2 * q + 1] = (__uint_as_float(h[q] & 0xffff0000u) + (__uint_as_float(m[q] & 0xffff0000u) + __uint_as_float(l[q] & 0xffff0000u))) *
                       (1.0f / kSplitScale);
    }
}

// Stores the four columns a lane holds of accumulator block nb to `dst` (which points at the
// lane's first column, 16 nb + 4 g), keeping to columns below w: 16-byte pieces, at whatever element
// they begin, and the columns of a block that w cuts one by one.
template <typename T>
__device__ __forceinline__ void store_acc4(T *dst, const typename Tr<T>::Acc &a, int nb, int g, int w) {
    constexpr int V = Tr<T>::V;
    if (16 * nb + 16 <= w) {
#pragma unroll
        for (int h = 0; h < 4 / V; ++h) {
            T tmp[V];
#pragma unroll
            for (int i = 0; i < V; ++i) tmp[i] = a[V * h + i];
            store_any<T, V>(dst + V * h, tmp);
        }
    } else {
#pragma unroll
        for (int h = 0; h < 4 / V; ++h) {
            const int col = 16 * nb + 4 * g + V * h;
            if (col + V <= w) {
                T tmp[V];
#pragma unroll
                for (int i = 0; i < V; ++i) tmp[i] = a[V * h + i];
                store_any<T, V>(dst + V * h, tmp);
            } else {
#pragma unroll
                for (int i = 0; i + 1 < V; ++i)
                    if (col + i < w) dst[V * h + i] = a[V * h + i];
            }
        }
    }
}

__device__ __forceinline__ int pow2_at_least(int x) {
    int g = 1;
    while (g < x) g <<= 1;
    return g;
}

template <typename T> constexpr int dtype_of() { return sizeof(T) == 8 ? TF_F64 : TF_F32; }

extern __shared__ __align__(16) unsigned char tf_smem[];

// ------------------------------------------------------------------------------------------ host

template <typename K> int raise_lds_limit(K kernel, int64_t bytes) {
    return (int)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Workgroups of a kernel that one compute unit holds at once (registers and LDS), 1..most.
template <typename K> int resident_per_cu(K kernel, int threads, int64_t lds_bytes, int most) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void *>(kernel),
                                                     threads, (size_t)lds_bytes) != hipSuccess)
        nb = 1;
    return nb < 1 ? 1 : (nb > most ? most : nb);
}

}  // namespace
}  // namespace tf
