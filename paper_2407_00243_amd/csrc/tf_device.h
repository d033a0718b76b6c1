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
