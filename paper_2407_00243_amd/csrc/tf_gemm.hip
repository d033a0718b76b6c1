// D1 = B C in fp32 on the bf16 matrix cores (gemm_splits; other products: k_gemm in tf_kernels.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "tf_device.h"

namespace tf {
namespace {

// A wave multiplies blocks of 32 rows of B (two blocks of sixteen, so that what is read of C from LDS is used twice: its
// reads then take half of what the LDS delivers).  C sits in LDS in three parts (split_pair), in operand order: per step of
// 32 k, per block of sixteen columns, per part sixteen bytes for each lane.  Rows of B are split as their step comes, and the
// same step of the wave's next block is fetched into the registers that this frees: a block's loads are on their way for as
// long as a block is multiplied, ahead of its stores, which they do not wait for.  More than four blocks of columns take two
// turns, with the rows split twice: the two sums of all of them leave no registers for the rows on their way (parts of all steps
// kept instead, two blocks of columns at a time, all loads together: n = 300000, 64 -> 64, the product alone 42.5 us, so 37.1;
// 128 -> 64 38.8 / 32.0; 96 -> 96 70 / 71; n = 2^20, 128 -> 128 290 / 302).
//
// Lane group g = lane / 16 holds of step s the elements k = 32 s + 4 g + {0 .. 3} and 32 s + 16 + 4 g + {0 .. 3} of its rows
// (four lanes fetch 64 contiguous bytes); pieces of the last step that would reach past the row are moved back so that they
// end with it and put right when they have arrived.
//
// A block with a row outside the bound of the split (infinities, very large numbers) is multiplied again by the fp32
// instructions, which read B from memory and put C together from its parts.  Where a column of C is outside, C is put into
// LDS as it is, and all blocks go there alone (whole executions, R-MAT graph of 2^20 rows, 128 -> 128, us: within the bound 965, one
// column outside 1090, every row 1347, by k_gemm 1013; 2^17 rows, 64 -> 128, 68, 76, 90, 69).
//
// Bound by memory where columns are few; at 128 -> 128 the matrix cores are busy half of the time, behind loads, splits and
// stores of two waves.  us, first wavefronts, on the fp32 matrix cores / here: n = 2^20, 128 -> 128, 356 / 302; n = 150000, 128 -> 64,
// 37 / 32, 128 -> 41, 36 / 32; n = 300000, 96 -> 96, 87 / 71, 100 -> 50, 58 / 50; n = 40000, 64 -> 40, 12.1 / 9.2.  Lines of D1 and D
// are written whole and not in halves by two instructions (with six products in one sum, n = 2^20, 128 -> 128, 244 / 231; n =
// 131072, 64 -> 128, 32 / 29.5).  PASS: B passes through the caches without staying there (run_split), as rows of D that leave here do:
// what the gather that follows reads does stay.
constexpr int kRowRor8 = 0x128;      // DPP: rotate sixteen lanes by eight
__device__ __forceinline__ uint32_t other_half(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kRowRor8, 0xf, 0xf, false); }

template <int KD, int NB, bool PASS>
__global__ __launch_bounds__(kFusedThreads) void k_gemm_split(const GemmLaunch a) {
    static_assert(NB >= 2, "slices are of kSplitMinCols columns at least");
    typedef typename Piece16<float>::Vec Vec;
    const int slice = blockIdx.y;
    const int c0 = slice * a.cs;
    const int w = min(a.cs, a.ccol - c0), w_d1 = c0 + w < a.ccol ? w : a.d1_cols - c0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int g = lane >> 4, r = lane & 15;
    Word4 *Cl = reinterpret_cast<Word4 *>(tf_smem);
    uint32_t *cmax = reinterpret_cast<uint32_t *>(tf_smem + KD * NB * 3 * 1024);
    const float *__restrict__ B = static_cast<const float *>(a.B), *__restrict__ C = static_cast<const float *>(a.C);
    float *__restrict__ D1 = static_cast<float *>(a.D1), *__restrict__ D = static_cast<float *>(a.D);
    const uint32_t n = (uint32_t)a.n, nblk = (n + 31) >> 5;
    // contiguous range of row blocks per workgroup, waves interleaved inside it
    const uint32_t lb0 = (uint64_t)nblk * blockIdx.x / gridDim.x, lb1 = (uint64_t)nblk * (blockIdx.x + 1) / gridDim.x;

    // the last step's pieces: where they begin, as far as they are in the row
    int last[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) last[h] = min(32 * (KD - 1) + 16 * h + 4 * g, a.bcol - 4);
    Vec x[KD][2][2];
    auto row_of = [&](uint32_t lb, int i) __attribute__((always_inline)) { return min(lb * 32 + 16 * i + r, n - 1); };
    auto row_at = [&](uint32_t lb, int i) __attribute__((always_inline)) { return B + (uint64_t)row_of(lb, i) * (uint32_t)a.bcol; };
    auto load_step = [&](int s, const float *const(&brow)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const Vec *p = reinterpret_cast<const Vec *>(brow[i] + (s < KD - 1 ? 32 * s + 16 * h + 4 * g : last[h]));
                x[s][i][h] = PASS ? __builtin_nontemporal_load(p) : *p;
            }
    };

    // C: the first pieces of it are on their way before the first rows of B, and split while these are
    constexpr int NC = (KD * NB * 64 + kFusedThreads - 1) / kFusedThreads;
    float y[NC][8];
    auto load_c = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int e = e0 + u * (int)blockDim.x, l = e & 63, nb = (e >> 6) % NB, s = (e >> 6) / NB;
            const int col = 16 * nb + (l & 15), k = 32 * s + 4 * (l >> 4);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int kq = k + (q < 4 ? q : 12 + q);
                const bool in = kq < a.bcol && col < w && e < KD * NB * 64;
                y[u][q] = C[in ? (int64_t)kq * a.c_ldk + (int64_t)(c0 + col) * a.c_ldc : 0];
                if (!in) y[u][q] = 0.0f;
            }
        }
    };
    auto put_c_whole = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int e = e0 + u * (int)blockDim.x;
            if (e >= KD * NB * 64) break;
#pragma unroll
            for (int p = 0; p < 2; ++p)
                Cl[((e >> 6) * 3 + p) * 64 + (e & 63)] = Word4{__float_as_uint(y[u][4 * p]), __float_as_uint(y[u][4 * p + 1]),
                                                               __float_as_uint(y[u][4 * p + 2]), __float_as_uint(y[u][4 * p + 3])};
        }
    };
    auto put_c = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int e = e0 + u * (int)blockDim.x, l = e & 63, nb = (e >> 6) % NB;
            if (e >= KD * NB * 64) break;
            uint32_t most = 0;      // (bits: a NaN counts as more than infinity)
            Word4 part[3];
#pragma unroll
            for (int q = 0; q < 8; q += 2) {
                most = max(most, max(__float_as_uint(y[u][q]) & 0x7fffffffu, __float_as_uint(y[u][q + 1]) & 0x7fffffffu));
                split_pair(part, q / 2, y[u][q], y[u][q + 1]);
            }
            atomicMax(&cmax[16 * nb + (l & 15)], most);
#pragma unroll
            for (int p = 0; p < 3; ++p) Cl[((e >> 6) * 3 + p) * 64 + l] = part[p];
        }
    };
    load_c(threadIdx.x);
    uint32_t lb = lb0 + wave;
    {
        const float *brow[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) brow[i] = row_at(lb, i);
#pragma unroll
        for (int s = 0; s < KD; ++s) load_step(s, brow);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int i = threadIdx.x; i < NB * 16; i += blockDim.x) cmax[i] = 0;
    __syncthreads();
    put_c(threadIdx.x);
    for (int e0 = (int)threadIdx.x + NC * (int)blockDim.x; e0 < KD * NB * 64; e0 += NC * (int)blockDim.x) {
        load_c(e0);
        put_c(e0);
    }
    __syncthreads();
    bool c_bad;
    const float row_bound = split_row_bound(cmax, NB * 16, lane, c_bad);
    if (c_bad) {      // (all waves of the workgroup; C as it is in the place of its parts)
        for (int e0 = (int)threadIdx.x; e0 < KD * NB * 64; e0 += NC * (int)blockDim.x) {
            load_c(e0);
            put_c_whole(e0);
        }
        __syncthreads();
    }

    // pieces of the last step that were moved back
    auto set_right = [&](Vec &x, int h) __attribute__((always_inline)) {
        const int back = 32 * (KD - 1) + 16 * h + 4 * g - last[h];
        Vec t;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            t[q] = 0.0f;
#pragma unroll
            for (int j = q; j < 4; ++j)
                if (back == j - q) t[q] = x[j];
        }
        x = t;
    };
    // (without info words any words are read: a load behind a branch is waited for there)
    const uint32_t *infos = a.row_info ? a.row_info : static_cast<const uint32_t *>(a.B);
    const float *scales = a.row_scale ? static_cast<const float *>(a.row_scale) : B;
    for (; lb < lb1; lb += nwaves) {
        // (the reads of C stay in the loop: in registers they would not fit)
        asm volatile("" ::: "memory");
        uint32_t info[2];
        float scale[2];
        const float *brow[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            info[i] = infos[row_of(lb, i)];
            scale[i] = scales[row_of(lb, i)];
            brow[i] = row_at(lb + nwaves, i);
        }
        bool fp32 = c_bad;
        // N blocks of columns from NB0 on: products and stores
        auto columns = [&](auto n_c, auto nb0_c) __attribute__((always_inline)) {
            constexpr int N = decltype(n_c)::value, NB0 = decltype(nb0_c)::value;
            constexpr bool FIRST = NB0 == 0, LAST = NB0 + N == NB;
            floatx4 acc[2][N];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < N; ++j) acc[i][j] = floatx4{0, 0, 0, 0};
            if (!c_bad) {
                floatx4 small[2][N];
                float most[2] = {0.0f, 0.0f};
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < N; ++j) small[i][j] = floatx4{0, 0, 0, 0};
#pragma unroll
                for (int s = 0; s < KD; ++s) {
                    if (FIRST && s == KD - 1 && a.bcol != 32 * KD) {
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int i = 0; i < 2; ++i) set_right(x[s][i][h], h);
                    }
                    Word4 part[2][3];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int q = 0; q < 4; q += 2) {
                                if constexpr (FIRST) most[i] = fmaxf(fmaxf(most[i], fabsf(x[s][i][h][q])), fabsf(x[s][i][h][q + 1]));
                                split_pair(part[i], 2 * h + q / 2, x[s][i][h][q], x[s][i][h][q + 1]);
                            }
                    // (the next block's loads after the last split, whose registers they take, and ahead of the multiplications)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        asm volatile("" : "+v"(most[i]));
#pragma unroll
                        for (int p = 0; p < 3; ++p) asm volatile("" : "+v"(part[i][p]));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (LAST) load_step(s, brow);
                    __builtin_amdgcn_sched_barrier(0);
                    // (one address a step: what lies past 64 KiB would have a register for every block, kept outside of the loop)
                    int at_step = s * (NB * 3 * 64) + lane;
                    if constexpr (KD * NB * 3 > 64) asm volatile("" : "+v"(at_step));
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        const Word4 *at = Cl + (at_step + (NB0 + j) * 3 * 64);
                        const Word4 c[3] = {at[0], at[64], at[128]};
                        auto multiply = [&](floatx4(&sums)[2][N], int cp, int bp) __attribute__((always_inline)) {
#pragma unroll
                            for (int i = 0; i < 2; ++i) sums[i][j] = mfma16_bf16(c[cp], part[i][bp], sums[i][j]);
                        };
                        multiply(small, 2, 1);
                        multiply(acc, 0, 0);
                        multiply(small, 1, 2);
                        multiply(small, 2, 0);
                        multiply(small, 0, 2);
                        multiply(small, 1, 1);
                        multiply(small, 1, 0);
                        multiply(small, 0, 1);
                    }
                }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < N; ++j) acc[i][j] = split_sum(acc[i][j], small[i][j]);
                if constexpr (FIRST) {
                    bool bad = false;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        asm volatile("" : "+v"(info[i]), "+v"(scale[i]));      // (here, not where they are fetched)
                        float m = fmaxf(most[i], __shfl_xor(most[i], 16, 64));
                        m = fmaxf(m, __shfl_xor(m, 32, 64));
                        // (rows that are not stored may hold anything)
                        const bool used = !a.row_info || (info[i] & (kInfoSpill | kInfoDirect));
                        bad |= used && split_exceeds(m, row_bound);
                    }
                    fp32 = __builtin_amdgcn_ballot_w64(bad) != 0;
                }
            }
            if (fp32) {
                const float *row[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) row[i] = row_at(lb, i);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < N; ++j) acc[i][j] = floatx4{0, 0, 0, 0};
#pragma unroll 1
                for (int s = 0; s < KD; ++s) {
                    Vec b[2][2];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            b[i][h] = *reinterpret_cast<const Vec *>(row[i] + (s < KD - 1 ? 32 * s + 16 * h + 4 * g : last[h]));
                            if (s == KD - 1 && a.bcol != 32 * KD) set_right(b[i][h], h);
                        }
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        float c[8];
                        split_whole(c, Cl + (s * NB + NB0 + j) * 3 * 64 + lane, c_bad);
#pragma unroll
                        for (int q = 0; q < 8; ++q)
#pragma unroll
                            for (int i = 0; i < 2; ++i) acc[i][j] = mfma16(c[q], b[i][q / 4][q % 4], acc[i][j]);
                    }
                }
            }
            // Two blocks of columns leave together, eight rows at a time, so that an instruction writes whole lines of 128 bytes: a
            // lane changes places with the one eight rows on.
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t row0 = lb * 32 + 16 * i;
                const uint32_t ri = row0 + r < n ? d1_info(a.row_info != nullptr, info[i]) : 0u, rx = other_half(ri);
                const float scale_x = __uint_as_float(other_half(__float_as_uint(scale[i])));
                // (to_d1: rows of the workspace, else of D)
                auto store = [&](auto to_d1) __attribute__((always_inline)) {
                    constexpr bool TO_D1 = decltype(to_d1)::value;
                    constexpr uint32_t kinds = TO_D1 ? kInfoSpill : kInfoDirect | kInfoZero;
                    if (__builtin_amdgcn_ballot_w64((ri & kinds) != 0) == 0) return;
                    const int ws = TO_D1 ? w_d1 : w;
                    auto row_start = [&](uint32_t info, uint32_t row) __attribute__((always_inline)) {
                        if constexpr (TO_D1) return D1 + d1_slot(a.row_info != nullptr, info, row) * a.d1_sw + 4 * g;
                        else return D + (int64_t)row * a.ccol + c0 + 4 * g;
                    };
                    auto scaled = [&](floatx4 y, uint32_t info, float by) __attribute__((always_inline)) {
                        if constexpr (!TO_D1)
#pragma unroll
                            for (int v = 0; v < 4; ++v) y[v] = info & kInfoZero ? 0.0f : by * y[v];
                        return y;
                    };
                    auto at_col = [&](int nb) __attribute__((always_inline)) {
                        const int cb = c0 + 16 * nb;        // the workspace is cut into slices of d1_sw columns
                        return TO_D1 ? (int64_t)(cb >> a.d1_sw_shift) * a.d1_slice_stride + (cb & a.d1_sw_mask) : 16 * nb;
                    };
                    const bool low = r < 8;
                    const uint32_t r0 = low ? ri : rx, r1 = low ? rx : ri;
                    const float s0 = low ? scale[i] : scale_x, s1 = low ? scale_x : scale[i];
                    float *own = row_start(ri, row0 + r), *dst0 = row_start(r0, row0 + (r & 7)) + (low ? 0 : 16),
                          *dst1 = row_start(r1, row0 + 8 + (r & 7)) + (low ? 0 : 16);
#pragma unroll
                    for (int j = 0; j < N; j += 2) {
                        const int nb = NB0 + j;
                        const bool pair = j + 1 < N && 16 * nb + 32 <= ws && (!TO_D1 || ((c0 + 16 * nb) & a.d1_sw_mask) + 32 <= a.d1_sw);
                        if (pair) {
                            floatx4 y0, y1;
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int lo = __float_as_int(acc[i][j][v]), hi = __float_as_int(acc[i][j + 1 < N ? j + 1 : j][v]);
                                y0[v] = __int_as_float(__builtin_amdgcn_update_dpp(lo, hi, kRowRor8, 0xf, 0xc, false));
                                y1[v] = __int_as_float(__builtin_amdgcn_update_dpp(hi, lo, kRowRor8, 0xf, 0x3, false));
                            }
                            typedef typename Piece16<float>::Vec Vec;
                            auto put = [&](float *to, const Vec &y) __attribute__((always_inline)) {
                                if constexpr (TO_D1) *reinterpret_cast<Vec *>(to) = y;
                                else __builtin_nontemporal_store(y, reinterpret_cast<Vec *>(to));
                            };
                            if (r0 & kinds) put(dst0 + at_col(nb), scaled(y0, r0, s0));
                            if (r1 & kinds) put(dst1 + at_col(nb), scaled(y1, r1, s1));
                        } else if (ri & kinds) {
                            store_acc4<float>(own + at_col(nb), scaled(acc[i][j], ri, scale[i]), nb, g, ws);
                            if (j + 1 < N) store_acc4<float>(own + at_col(nb + 1), scaled(acc[i][j + 1 < N ? j + 1 : j], ri, scale[i]), nb + 1, g, ws);
                        }
                    }
                };
                store(std::true_type());
                store(std::false_type());
            }
        };
        // (four blocks at a time: registers for their two sums, rows of B and the next ones)
        constexpr int N0 = NB < 4 ? NB : 4;
        columns(std::integral_constant<int, N0>(), std::integral_constant<int, 0>());
        if constexpr (NB > N0) columns(std::integral_constant<int, NB - N0>(), std::integral_constant<int, N0>());
    }
}

// ------------------------------------------------------------------------------------------ host

template <int KD, int NB, bool PASS> int run_split2(const GemmLaunch &a, hipStream_t st) {
    constexpr int64_t lds = split_lds_bytes(KD, NB);
    const int64_t nblk = (a.n + 31) / 32;
    constexpr int nwaves = kFusedThreads / 64;
    static std::mutex m;
    static int occ = 0;
    int wg_per_cu;
    {
        std::lock_guard<std::mutex> lock(m);
        if (!occ) {
            const int e = raise_lds_limit(k_gemm_split<KD, NB, PASS>, lds);
            if (e) return e;
            occ = resident_per_cu(k_gemm_split<KD, NB, PASS>, 64 * nwaves, lds, 16);
        }
        wg_per_cu = occ;
    }
    // as many workgroups as the machine holds at once
    const int64_t most = std::max<int64_t>(1, (int64_t)a.n_cu * wg_per_cu / a.n_slices);
    const int64_t gx = std::min(most, (nblk + nwaves - 1) / nwaves);
    (void)hipGetLastError();
    k_gemm_split<KD, NB, PASS><<<dim3((unsigned)gx, (unsigned)a.n_slices), dim3(64 * nwaves), lds, st>>>(a);
    return (int)hipGetLastError();
}
// Rows of B pass through the caches without staying there where what is written is more than the L2s hold, which the launch that
// follows gathers from, and rows of B are whole lines, or a line that a load takes a part of is gone when the next one comes for the
// rest (100 -> 100, 150000 rows, 152 us passing, 142 staying).  What decides below 256 MB of B, D1 and D is whether the program has used
// the same operands just before, which only it knows; the rule takes those that come anew.  Whole executions on R-MAT graphs,
// us, staying / passing, three sets of operands in turn and, in brackets, one set again and again: 150000 rows, 128 -> 41 83.3 / 75.4
// (69.2 / 75.6), 128 -> 64 79.2 / 73.4 (68.2 / 73.1), 64 -> 64 69.5 / 63.7 (60.0 / 63.2), 96 -> 96 100.5 / 100.8 (90.5 / 98.0), 100000, 128 -> 128 99.5 /
// 92.1 (87.5 / 91.1), 70000, 128 -> 128 70.5 / 68.8 (66.0 / 69.4), 300000, 64 -> 64 129 / 131 (119 / 119), 128 -> 128 277 / 265 (275 / 263), 10^6,
// 64 -> 32 262 / 254 (261 / 256).  Not where the product is the second operation (D1 is D): what it reads was just written, and no
// launch follows (131072 rows, 64 -> 128 63.6 / 67.7, 300000, 32 -> 64 75.8 / 86.6, 10^6, 64 -> 128 663 / 683).
template <int KD, int NB> int run_split(const GemmLaunch &a, hipStream_t st) {
    const bool pass = a.D1 != a.D && a.bcol % 32 == 0 && a.n * a.d1_cols * 4 >= ((int64_t)32 << 20);
    if (pass) return run_split2<KD, NB, true>(a, st);
    return run_split2<KD, NB, false>(a, st);
}

template <int KD> int run_split_nb(const GemmLaunch &a, hipStream_t st) {
    switch (split_col_blocks(a.cs)) {
        case 2: return run_split<KD, 2>(a, st);
        case 3: return run_split<KD, 3>(a, st);
        case 4: return run_split<KD, 4>(a, st);
        case 6: return run_split<KD, 6>(a, st);
        case 8: return run_split<KD, 8>(a, st);
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace

int launch_gemm_split(const GemmLaunch &a, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch ((a.bcol + 31) / 32) {
        case 1: return run_split_nb<1>(a, st);
        case 2: return run_split_nb<2>(a, st);
        case 3: return run_split_nb<3>(a, st);
        case 4: return run_split_nb<4>(a, st);
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace tf
