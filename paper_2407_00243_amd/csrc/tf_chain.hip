// The chain D = A (B C) with a dense B in one pass over A:  D = (A B) C.
//
// A wave owns sixteen (virtual) rows of A at a time.  Four neighbouring lanes gather the rows of B of
// one of them, 64 contiguous bytes per load, and sum them up in registers; the sums change lanes
// through LDS into the layout that the matrix cores take as an operand, are multiplied by C, whose
// operands sit in LDS, and leave as sixteen rows of D.  Nothing of the product travels through
// memory: A, B and C are read, D is written, and there is one launch.
//
// (Gathering straight into the operand layout -- lane 16 g + r holding row r -- needs no exchange, but
// there four neighbouring lanes name four different rows, and the vector memory path merges
// neighbours only: 5.3 TB/s of gathered data whatever the cache hits, 2D stencil 64 -> 64 in 62 us.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "tf_device.h"

namespace tf {
namespace {

// Flags word of a buffer descriptor for plain 32-bit data (range-checked byte offsets).
constexpr int kBufferRaw = 0x00020000;

// D is not read again here: its stores pass through the L2 without staying there (2D stencil, fp32
// 64 -> 64, n = 2^18: 53 us with plain stores, 40 us).
constexpr int kNonTemporal = 2;

// Stages all of C in LDS in the order the multiplications take it: per group of NBC blocks of
// sixteen columns, per k step i = s V + q, per block nb: 64 elements, lane l's being
// C[KC s + V (l / 16) + q][16 (NBC group + nb) + column l % 16 of the block], zero beyond bCol.  The
// columns of a block are taken in an order that leaves the four results of lane (g, r) as columns 4 g
// .. 4 g + 3 in fp32 and 2 g, 2 g + 1, 8 + 2 g, 9 + 2 g in fp64: whole 16-byte pieces.  The columns
// come in pieces of V (16 bytes of D); a piece that would reach past cCol is moved back so that it
// ends there, and so is its store: what it shares with the piece before is computed and stored twice.
// Pieces p0 + u * blockDim.x of C, u < kStageC: load_c fetches them, write_c puts them into LDS.  A piece
// is sixteen bytes along a row of C as it is stored: V columns of one k, or, transposed, V values of
// k of one column.  Pieces that would reach past the row's end are moved back like those of B, in
// registers here (the elements they then miss are zeros).
constexpr int kStageC = 8;
template <typename T> struct CPiece {
    typename Piece16<T>::Vec x;
    int at;                // LDS position of its first element, -1: none
};
template <typename T, int KS, int NBC, bool CT>
__device__ __forceinline__ void load_c(CPiece<T> (&tmp)[kStageC], int p0, int total, int groups,
                                       int col0, const ChainLaunch &a) {
    constexpr int V = Tr<T>::V, KC = 4 * V;
    typedef typename Piece16<T>::Vec Vec;
    const T *__restrict__ C = static_cast<const T *>(a.C);
#pragma unroll
    for (int u = 0; u < kStageC; ++u) {
        const int p = p0 + u * (int)blockDim.x;
        tmp[u].at = -1;
        tmp[u].x = Vec{};
        if (p >= total) continue;
        if constexpr (!CT) {
            // p -> (k, block of columns, piece of the block)
            const int w = p % (16 / V), rest = p / (16 / V), nbt = rest % (groups * NBC), k = rest / (groups * NBC);
            const int i = k / KC * V + k % V, g = k / V % 4;
            // columns 4 w .. of fp32 are m = 4 w ..; columns 2 w, 2 w + 1 of fp64 m = 8 (w / 4) + w % 4 + {0, 4}
            const int m = V == 4 ? 4 * w : 8 * (w / 4) + w % 4;
            tmp[u].at = ((nbt / NBC * (KS * V) + i) * NBC + nbt % NBC) * 64 + 16 * g + m;
            const int col = min(col0 + 16 * nbt + V * w, a.ccol - V);
            if (k < a.bcol) tmp[u].x = *reinterpret_cast<const Vec *>(C + (int64_t)k * a.ccol + col);
        } else {
            // p -> (column, piece of k)
            const int kp = p % (4 * KS), c = p / (4 * KS), nbt = c / 16, cc = c % 16;
            const int m = V == 4 ? cc : 8 * (cc / 8) + cc % 8 / 2 + 4 * (cc % 2);
            tmp[u].at = ((nbt / NBC * (KS * V) + kp / 4 * V) * NBC + nbt % NBC) * 64 + 16 * (kp % 4) + m;
            const int cw = col0 + c / V * V, col = min(cw, a.ccol - V) + c % V;
            const int back = max(0, V * kp - (a.bcol - V));
            const Vec y = *reinterpret_cast<const Vec *>(C + (int64_t)col * a.bcol + (V * kp - back));
#pragma unroll
            for (int q = 0; q < V; ++q)
#pragma unroll
                for (int j = q; j < V; ++j)
                    if (back == j - q) tmp[u].x[q] = y[j];
        }
    }
}
template <typename T, int NBC, bool CT>
__device__ __forceinline__ void write_c(T *Cl, const CPiece<T> (&tmp)[kStageC]) {
    constexpr int V = Tr<T>::V;
#pragma unroll
    for (int u = 0; u < kStageC; ++u) {
        if (tmp[u].at < 0) continue;
#pragma unroll
        for (int q = 0; q < V; ++q) Cl[tmp[u].at + (CT ? q * NBC * 64 : V == 4 ? q : 4 * q)] = tmp[u].x[q];
    }
}

// KS: 16-byte pieces per lane of a row of B (bCol <= 4 V KS), NBC: blocks of sixteen columns of D
// multiplied at a time.
//
// A block's entries are gathered in passes of up to EM entries per row.  Order of a wave's work per
// block: add up the first pass (in flight since the block before), gather and add up the others,
// send out the first gathers of the next block, and only then multiply and store.  Loads and stores
// of a wave complete in order on this machine, so gathers that were sent out after the stores of D
// would wait for these to reach memory.
template <typename T, int KS, int NBC>
__global__ __launch_bounds__(kChainThreads, chain_waves(dtype_of<T>(), KS, NBC)) void k_gather_gemm(
    const ChainLaunch a, const ChainBlock *__restrict__ blocks, const int32_t *__restrict__ rows,
    const int32_t *__restrict__ idx, const T *__restrict__ val, const char *__restrict__ B,
    void *D) {
    constexpr int V = Tr<T>::V, KC = 4 * V;
    constexpr int EM = chain_entries(KS);
    constexpr int K0 = chain_ksteps_below(dtype_of<T>(), KS);      // pieces that are whole for certain
    typedef typename Piece16<T>::Vec Vec;
    typedef T Vec16 __attribute__((ext_vector_type(V)));
    typedef const __attribute__((address_space(1))) char *GlobalBytes;
    typedef const __attribute__((address_space(1))) Vec *GlobalVec;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = (int)blockDim.x >> 6;
    const int g = lane >> 4, r = lane & 15;              // as the matrix cores see the lane
    // as it gathers: LR lanes share a row (128 contiguous bytes of it per load when rows are that long),
    // 64 / LR rows at a time, RS times; piece P = pp + LR t of the rows rr + 64 h / LR
    constexpr int LR = KS % 2 == 0 ? 8 : 4, RS = LR / 4, KP = KS / RS;
    const int pp = lane % LR, rr = lane / LR;
    T *Cl = reinterpret_cast<T *>(tf_smem);
    // the column groups of this workgroup (all of them, unless the launch has few blocks of rows)
    const int g0 = (int)blockIdx.y * a.groups_per_wg;
    const int groups = min(a.groups_per_wg, a.n_groups - g0), col0 = g0 * NBC * 16;
    // behind C, per wave: the place where pieces change lanes -- sums into operands (TS x 16 rows x 64
    // bytes; the pieces of a row are swizzled so that the sixteen rows' pieces g sit in different
    // banks), results into rows of D (16 rows of CB blocks and 16 bytes) -- then the offsets of the
    // rows of D and the entries of a pass (NE x 64 values, then addresses of rows of B)
    constexpr int NE = chain_entry_loads(KS), TS = chain_exchange(KS), CB = chain_store_blocks(dtype_of<T>(), KS, NBC);
    constexpr int W = CB * 16 / V, PITCH = W * 16 + 16;
    unsigned char *ex = tf_smem + a.groups_per_wg * (NBC * KS * V * 64 * (int)sizeof(T)) +
                        wave * (int)chain_wave_lds(dtype_of<T>(), KS, NBC);
    uint32_t *er = reinterpret_cast<uint32_t *>(ex + chain_exchange_bytes(dtype_of<T>(), KS, NBC));
    T *ev = reinterpret_cast<T *>(er + 16);
    uint64_t *ea = reinterpret_cast<uint64_t *>(ev + NE * 64);
    const unsigned char *ex_r = ex + r * 64 + (g ^ (r >> 2)) * 16;

    // blocks of this wave: every XCD has a contiguous range, through which its waves move side by side
    // (rows of B that neighbouring blocks share stay in that XCD's L2); wide rows: after a.whole_rounds the blocks
    // that are left are dealt over the workgroups (narrow ones gain 5 % at most, and lose up to 4 to the longer
    // start: bands of 15204 rows, fp32 19 -> 16, 8.8 -> 9.1 us)
    const int per = (a.n_blocks + kXcds - 1) / kXcds, xcd = blockIdx.x % kXcds, wg = (int)(blockIdx.x / kXcds);
    const int end = min(a.n_blocks, (xcd + 1) * per), n_wg = (int)(gridDim.x / kXcds), step = n_wg * nwaves;
    auto block_after = [&](int b) __attribute__((always_inline)) {
        if constexpr (KS < kChainSpreadDepth) return b + step;
        const int dealt = xcd * per + a.whole_rounds * step;
        return b + step < dealt ? b + step : b < dealt ? dealt + wave * n_wg + wg : end;
    };
    int blk = xcd * per + wg * nwaves + wave;

    // The entries of a pass: fetched a pass ahead, 64 (four slots of sixteen rows) per load, put into
    // LDS when their turn comes, read back by the lanes of their row.  A column becomes the address of its
    // row of B on the way (once per entry, not once per lane and gather), padding that of zeros: whatever B
    // holds, padding adds nothing.  The waves of an XCD use different copies of the zeros, and have theirs
    // in the L1 before the first gather needs it (band of 4096 rows, fp64 32 -> 32: 6.24 us with one copy, 6.15
    // with sixteen, 5.90 with sixteen fetched ahead; 5.98 when padding read the row's last column again).
    const uint32_t row_bytes = (uint32_t)a.bcol * (uint32_t)sizeof(T);
    const uint64_t zeros = reinterpret_cast<uint64_t>(a.zeros) +
                           (blockIdx.x / kXcds * nwaves + wave) % kChainZeroRows * kChainRowBytes;
    const float zeros_ahead = *(const __attribute__((address_space(1))) float *)(zeros + min((uint32_t)lane * 16, row_bytes - 4));
    int32_t ci[NE];
    T vi[NE];
    auto fetch = [&](uint32_t slot) __attribute__((always_inline)) {
        const int64_t at = (int64_t)slot * 16 + lane;
#pragma unroll
        for (int e = 0; e < NE; ++e) ci[e] = idx[at + e * 64];
#pragma unroll
        for (int e = 0; e < NE; ++e) vi[e] = val[at + e * 64];
    };
    auto put = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const uint64_t at = reinterpret_cast<uint64_t>(B) + (uint64_t)(uint32_t)ci[e] * row_bytes;
            // (all ones for padding; kept from the compiler, which would make a branch of the choice)
            int32_t pad = ci[e] >> 31;
            asm("" : "+v"(pad));
            ea[e * 64 + lane] = at ^ ((at ^ zeros) & (uint64_t)(int64_t)pad);
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) ev[e * 64 + lane] = vi[e];
        __builtin_amdgcn_wave_barrier();
    };
    // row of D behind the lane's (virtual) row
    auto row_id = [&](const ChainBlock &b) __attribute__((always_inline)) {
        return rows[b.row_begin + min(r >> (b.info & 7), (b.info >> 7) - 1)];
    };
    ChainBlock d{}, dn{};
    int32_t row = 0, row_n = 0;
    if (blk < end) {
        d = blocks[blk];
        row = row_id(d);
        fetch(d.slot_base);
        dn = blocks[min(block_after(blk), end - 1)];
    }
    // pieces of a row of B that may reach past bCol are moved back so that they end with the row, and put
    // right after the sums are complete
    constexpr int T0 = K0 / RS;                          // pieces t below are whole
    // (offsets in bytes, one addition per load: in rows with a whole piece the others from there, else from the
    // row's start; band of 15204 rows of 41, fp32 19 -> 16, 8.95 -> 8.58 us)
    const int first = T0 > 0 ? pp * 16 : 0;
    int64_t moved[KP - T0];
#pragma unroll
    for (int t = T0; t < KP; ++t)
        moved[t - T0] = min(V * (pp + LR * t), a.bcol - V) * (int)sizeof(T) - first;

    typedef uint32_t Word4 __attribute__((ext_vector_type(4)));
    const auto Dr = __builtin_amdgcn_make_buffer_rsrc(D, 0, (uint32_t)(a.n * a.ccol * (int64_t)sizeof(T)),
                                                      kBufferRaw);

    Vec x[EM][RS][KP];
    T acc[RS][KP][V];
    // (n is wave-uniform: a branch per entry)
    auto issue = [&](int n) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < EM; ++e) {
            if (e < n) {
#pragma unroll
                for (int h = 0; h < RS; ++h) {
                    const GlobalBytes p = (GlobalBytes)(ea[e * 16 + rr + h * (64 / LR)] + first);
#pragma unroll
                    for (int t = 0; t < KP; ++t)
                        x[e][h][t] = *(GlobalVec)(t < T0 ? p + 16 * LR * t : p + moved[t < T0 ? 0 : t - T0]);
                }
            }
        }
    };
    auto consume = [&](int n) __attribute__((always_inline)) {
        // All values first: one trip to LDS and back, not one per entry behind its branch (band of 15204 rows of
        // 41, fp32 19 -> 16, 9.76 -> 8.95 us; slots beyond the pass are read too, and not used).
        T w[EM][RS];
#pragma unroll
        for (int e = 0; e < EM; ++e)
#pragma unroll
            for (int h = 0; h < RS; ++h) w[e][h] = ev[e * 16 + rr + h * (64 / LR)];
#pragma unroll
        for (int e = 0; e < EM; ++e)
#pragma unroll
            for (int h = 0; h < RS; ++h) asm volatile("" : "+v"(w[e][h]));
#pragma unroll
        for (int e = 0; e < EM; ++e) {
            if (e < n) {
#pragma unroll
                for (int h = 0; h < RS; ++h) {
                    const T v = w[e][h];
#pragma unroll
                    for (int t = 0; t < KP; ++t)
#pragma unroll
                        for (int q = 0; q < V; ++q) acc[h][t][q] += v * x[e][h][t][q];
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto pass_len = [](const ChainBlock &b) { return (b.info >> 3) & 15; };
    auto first_count = [&](const ChainBlock &b) { return min(pass_len(b), b.slots); };

    // Start-up: the first gathers of the first block go out before C is put into LDS
    {
        const int total = groups * NBC * 16 * KS * 4;
        CPiece<T> tmp[kStageC];
        auto first_issue = [&]() __attribute__((always_inline)) {
            if (blk < end) {
                put();
                fetch(d.slots > pass_len(d) ? d.slot_base + pass_len(d) : dn.slot_base);
                issue(first_count(d));
            }
        };
        auto stage = [&](auto ct_c) __attribute__((always_inline)) {
            constexpr bool CT = decltype(ct_c)::value;
            load_c<T, KS, NBC, CT>(tmp, threadIdx.x, total, groups, col0, a);
            first_issue();
            write_c<T, NBC, CT>(Cl, tmp);
            for (int p0 = (int)threadIdx.x + kStageC * (int)blockDim.x; p0 < total;
                 p0 += kStageC * (int)blockDim.x) {
                load_c<T, KS, NBC, CT>(tmp, p0, total, groups, col0, a);
                write_c<T, NBC, CT>(Cl, tmp);
            }
        };
        if (a.c_transposed) stage(std::true_type());
        else stage(std::false_type());
        __syncthreads();
        if (blk >= end) return;
        __builtin_amdgcn_s_waitcnt(0);
        asm volatile("" : : "v"(zeros_ahead));
    }

    for (;;) {
        const int next = block_after(blk);
        const bool has_next = next < end;
        const ChainBlock dnn = blocks[min(block_after(next), end - 1)];
#pragma unroll
        for (int h = 0; h < RS; ++h)
#pragma unroll
            for (int t = 0; t < KP; ++t)
#pragma unroll
                for (int q = 0; q < V; ++q) acc[h][t][q] = T(0);
        const int len = pass_len(d);
        consume(first_count(d));
        for (int s0 = len; s0 < d.slots; s0 += len) {
            const int count = min(len, d.slots - s0);
            put();
            fetch(s0 + len < d.slots ? d.slot_base + s0 + len : dn.slot_base);
            issue(count);
            consume(count);
        }
        // the gathers of the next block (the last block sends those of some block out, for nothing)
        put();
        row_n = row_id(dn);
        fetch(dn.slots > pass_len(dn) ? dn.slot_base + pass_len(dn) : dnn.slot_base);
        issue(first_count(dn));
        __builtin_amdgcn_sched_barrier(0);

        // into the operand layout (a wave's LDS operations take effect in order)
        T f[KS][V];
#pragma unroll
        for (int s0 = 0; s0 < KS; s0 += TS) {
#pragma unroll
            for (int h = 0; h < RS; ++h)
#pragma unroll
                for (int t = s0 / RS; t < KP && t < (s0 + TS) / RS; ++t) {
                    const int P = pp + LR * t - 4 * s0, gr = rr + h * (64 / LR);
                    Vec16 y;
#pragma unroll
                    for (int q = 0; q < V; ++q) y[q] = acc[h][t][q];
                    *reinterpret_cast<Vec16 *>(ex + (P >> 2) * 1024 + gr * 64 + ((P & 3) ^ (gr >> 2)) * 16) = y;
                }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int s = s0; s < KS && s < s0 + TS; ++s) {
                const Vec16 y = *reinterpret_cast<const Vec16 *>(ex_r + (s - s0) * 1024);
#pragma unroll
                for (int q = 0; q < V; ++q) f[s][q] = y[q];
            }
            __builtin_amdgcn_wave_barrier();
        }
        // pieces that were moved back; elements past bCol are zeros
#pragma unroll
        for (int s = K0; s < KS; ++s) {
            const int b = max(0, KC * s + V * g - (a.bcol - V));
            T t[V];
#pragma unroll
            for (int q = 0; q < V; ++q) {
                t[q] = T(0);
#pragma unroll
                for (int j = q; j < V; ++j)
                    if (b == j - q) t[q] = f[s][j];
            }
#pragma unroll
            for (int q = 0; q < V; ++q) f[s][q] = t[q];
        }
        // the parts of a row that was cut up sit in adjacent lanes
        const int slog = d.info & 7, n_rows = d.info >> 7;
        for (int m = 1; m < (1 << slog); m <<= 1) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int q = 0; q < V; ++q) f[s][q] += __shfl_xor(f[s][q], m, 64);
        }
        // The rows of D leave through LDS so that neighbouring lanes store neighbouring pieces, up to 256
        // contiguous bytes of a row (straight from the matrix cores a store would cover 64 bytes of
        // each of sixteen rows: 7 to 13 % slower where D comes from or goes to memory).
        // Stores go through a buffer descriptor, and out-of-range lanes (virtual rows that are not the
        // first of their row, columns past cCol) name an offset beyond it, which the hardware drops:
        // without a branch around the stores the compiler knows how many are on their way, and its
        // wait for the next block's gathers, which were sent out before, does not include them.
        if (g == 0)
            er[r] = (r >> slog) < n_rows && (r & ((1 << slog) - 1)) == 0 ? (uint32_t)row * (uint32_t)a.ccol : ~0u;
        const bool empty = d.slots == 0;      // (empty rows are zeros whatever C holds)
        __builtin_amdgcn_s_setprio(0);
        int grp = 0;
        do {
            const T *Cg = Cl + grp * (NBC * KS * V * 64) + lane;
            typename Tr<T>::Acc o[NBC];
#pragma unroll
            for (int nb = 0; nb < NBC; ++nb) o[nb] = typename Tr<T>::Acc{0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < KS * V; ++i)
#pragma unroll
                for (int nb = 0; nb < NBC; ++nb)
                    o[nb] = mfma16(Cg[(i * NBC + nb) * 64], f[i / V][i % V], o[nb]);
#pragma unroll
            for (int nb0 = 0; nb0 < NBC; nb0 += CB) {
#pragma unroll
                for (int nb = nb0; nb < nb0 + CB; ++nb)
#pragma unroll
                    for (int h = 0; h < 4 / V; ++h) {
                        Vec16 y;
#pragma unroll
                        for (int q = 0; q < V; ++q) y[q] = empty ? T(0) : o[nb][V * h + q];
                        *reinterpret_cast<Vec16 *>(ex + r * PITCH + ((nb - nb0) * 16 / V + 4 * h + g) * 16) = y;
                    }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < W / 4; ++i) {
                    const int at = i * 64 + lane, sr = at / W, piece = at % W;
                    const int col = col0 + 16 * (grp * NBC + nb0) + piece * V;
                    const uint32_t row_off = er[sr];
                    const Word4 y = *reinterpret_cast<const Word4 *>(ex + sr * PITCH + piece * 16);
                    const uint32_t off = (row_off + (uint32_t)min(col, a.ccol - V)) * (uint32_t)sizeof(T);
                    __builtin_amdgcn_raw_buffer_store_b128(y, Dr, row_off != ~0u && col < a.ccol ? off : ~0u,
                                                           0, kNonTemporal);
                }
                __builtin_amdgcn_wave_barrier();
            }
        } while (++grp < groups);
        __builtin_amdgcn_s_setprio(3);
        if (!has_next) break;
        d = dn;
        dn = dnn;
        row = row_n;
        blk = next;
    }
}

// ------------------------------------------------------------------------------------------ host

struct ChainSetup {
    std::mutex m;
    int64_t raised = -1, occ_lds = -1;
    int occ_waves = 0, wg_per_cu = 1;
};

template <typename T, int KS, int NBC> int run_chain(ChainLaunch a, hipStream_t st) {
    static ChainSetup cs;
    auto kernel = k_gather_gemm<T, KS, NBC>;
    // A launch with few blocks of rows is spread over the machine by column groups too (the rows are then
    // gathered once per group, and a workgroup stages its part of C only): as far as the machine holds all
    // its waves at once, half of them where C is small and little is saved (us, all groups in one workgroup /
    // as chosen: bands of 17 entries, fp64 128 -> 128, n = 4096 34.3 / 21.4, 8192 40.7 / 27.5, 16384 40.9 /
    // 32.1; fp32 128 -> 128 20.1 / 11.8, 23.7 / 13.3, 23.8 / 18.9; with twice the waves 51.5 at n = 16384 in fp64,
    // 34.7 / 24.0 at 32768 in fp32; C of 32 KiB, fp64 32 -> 128, n = 16384, 12.0 / 11.1 with one group each).
    const int64_t group_lds = (int64_t)NBC * KS * Tr<T>::V * 64 * (int64_t)sizeof(T);
    const int64_t held = (int64_t)a.n_cu * (a.n_groups * group_lds <= 40 * 1024 ? 4 : 8);
    a.groups_per_wg = 1;
    while (a.n_blocks >= 2 * a.n_cu && a.groups_per_wg < a.n_groups &&
           (int64_t)a.n_blocks * ((a.n_groups + a.groups_per_wg - 1) / a.groups_per_wg) > held)
        ++a.groups_per_wg;
    const int n_y = (a.n_groups + a.groups_per_wg - 1) / a.groups_per_wg;
    const int64_t lds_c = a.groups_per_wg * group_lds;
    // Waves per workgroup: one copy of C per workgroup, so the more LDS it takes the more waves have
    // to share it; a launch with fewer blocks than the machine has room for is spread thin, as far
    // as a wave does not have to stage more than 8 KiB of C.
    int waves = lds_c <= 40 * 1024 ? 4 : 8;
    while (waves > 1 && (int64_t)a.n_blocks * n_y < (int64_t)a.n_cu * waves && waves * 4096 >= lds_c) waves /= 2;
    const int64_t lds = lds_c + waves * chain_wave_lds(a.dtype, KS, NBC);
    int wg_per_cu = 1;
    {
        std::lock_guard<std::mutex> lock(cs.m);
        if (lds > cs.raised) {
            const int e = raise_lds_limit(kernel, lds);
            if (e) return e;
            cs.raised = lds;
        }
        if (lds != cs.occ_lds || waves != cs.occ_waves) {
            cs.wg_per_cu = resident_per_cu(kernel, 64 * waves, lds, 16);
            cs.occ_lds = lds;
            cs.occ_waves = waves;
        }
        wg_per_cu = cs.wg_per_cu;
    }
    const int64_t want = ((int64_t)a.n_blocks + waves - 1) / waves;
    int64_t grid = std::min<int64_t>(want, (int64_t)a.n_cu * wg_per_cu);
    grid = (grid + kXcds - 1) / kXcds * kXcds;
    // Blocks of the last round, which does not take all waves: neighbouring blocks to neighbouring waves like the
    // others, or over all workgroups.  The latter where a workgroup fills a compute unit, which would have two blocks
    // for every wave while others have one (2D stencils, fp32 128 -> 128, 200^2 30.9 -> 24.9 us, 300^2 43.6 -> 42.8; fp64
    // 200^2 53.9 -> 44.8), and where the round is short.  Else neighbours: they share rows of B (3D stencil 60^3, fp32
    // 32 -> 32, 40 % of the waves, 17.8 us, 18.9 when spread).
    const int64_t wave_slots = grid / kXcds * waves, per = ((int64_t)a.n_blocks + kXcds - 1) / kXcds;
    const bool spread = waves == kChainThreads / 64 || per % wave_slots * 16 <= wave_slots;
    a.whole_rounds = (int32_t)(spread ? std::max<int64_t>(1, per / wave_slots) : per / wave_slots + 2);
    (void)hipGetLastError();      // an error left by an earlier, unrelated call is not this launch's
    kernel<<<dim3((unsigned)grid, (unsigned)n_y), dim3(64 * waves), lds, st>>>(
        a, a.blocks, a.rows, a.idx, static_cast<const T *>(a.vals), static_cast<const char *>(a.B), a.D);
    return (int)hipGetLastError();
}

template <typename T, int KS> int run_chain_nb(ChainLaunch a, hipStream_t st) {
    const int nb = (a.ccol + 15) / 16, nbc = chain_col_blocks(KS, a.ccol);
    a.n_groups = (nb + nbc - 1) / nbc;
    switch (nbc) {
        case 1: return run_chain<T, KS, 1>(a, st);
        case 2: return run_chain<T, KS, 2>(a, st);
    }
    if constexpr (KS < 16) return nbc == 3 ? run_chain<T, KS, 3>(a, st) : run_chain<T, KS, 4>(a, st);
    return (int)hipErrorInvalidValue;
}

}  // namespace

int launch_chain(const ChainLaunch &a, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (a.n_blocks == 0) return 0;
    const int ks = chain_ksteps(a.dtype, a.bcol);
    if (a.dtype == TF_F32) {
        switch (ks) {
            case 1: return run_chain_nb<float, 1>(a, st);
            case 2: return run_chain_nb<float, 2>(a, st);
            case 3: return run_chain_nb<float, 3>(a, st);
            case 4: return run_chain_nb<float, 4>(a, st);
            case 6: return run_chain_nb<float, 6>(a, st);
            case 8: return run_chain_nb<float, 8>(a, st);
        }
    } else {
        switch (ks) {
            case 2: return run_chain_nb<double, 2>(a, st);
            case 4: return run_chain_nb<double, 4>(a, st);
            case 6: return run_chain_nb<double, 6>(a, st);
            case 8: return run_chain_nb<double, 8>(a, st);
            case 12: return run_chain_nb<double, 12>(a, st);
            case 16: return run_chain_nb<double, 16>(a, st);
        }
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace tf
