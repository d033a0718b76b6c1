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

// fp32 on the bf16 matrix cores: C in three parts (split_pair), per group of NBC blocks of sixteen columns, per step s of
// 32 k, per block, per part sixteen bytes for each lane l, C[32 s + {0, 16} + 4 (l / 16) + {0 .. 3}][column l % 16 of the
// block]; elements past bCol are zeros.  An item is what four neighbouring lanes take: eight k of four columns, fetched by
// eight loads of sixteen bytes (element by element: band of 20011 rows of 11, 64 -> 64, 9.5 us, so 8.5).  KS2: steps; CT: C
// is transposed, its rows bCol long, else ld long; a piece of four columns that would reach past `cols` is moved back so
// that it ends there.
struct SplitC {
    const float *C;      // at the first column
    int ld, bcol, cols;
};
template <int KS2, bool CT>
__device__ __forceinline__ void load_split(floatx4 (&y)[8], const SplitC &c, int item, int total) {
    typedef typename Piece16<float>::Vec Vec;
    const int w = item & 3, g = item >> 2 & 3, s = (item >> 4) % KS2, nbt = (item >> 4) / KS2;
    const int col = min(16 * nbt + 4 * w, c.cols - 4);
#pragma unroll
    for (int q = 0; q < 8; ++q) y[q] = floatx4{0, 0, 0, 0};
    if (item >= total) return;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        // row of C as it is stored, first element in it, elements of the row
        const int k = 32 * s + 4 * g + (CT ? 16 * (q / 4) : q < 4 ? q : 12 + q);
        const int row = CT ? col + q % 4 : k, at = CT ? k : col, end = CT ? c.bcol : c.cols;
        if (row >= (CT ? c.cols : c.bcol)) continue;
        const float *p = c.C + (int64_t)row * (CT ? c.bcol : c.ld) + at;
        if (at + 4 <= end) {
            y[q] = *reinterpret_cast<const Vec *>(p);
        } else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (at + j < end) y[q][j] = p[j];
        }
    }
}
// Puts an item into LDS and the largest number (bits: a NaN counts as more than infinity) of each column into cmax.
template <int KS2, int NBC, bool CT>
__device__ __forceinline__ void write_split(Word4 *Cl, uint32_t *cmax, const floatx4 (&y)[8], int item, int total) {
    const int w = item & 3, g = item >> 2 & 3, s = (item >> 4) % KS2, nbt = (item >> 4) / KS2;
    if (item >= total) return;
    Word4 *to = Cl + ((nbt / NBC * KS2 + s) * NBC + nbt % NBC) * 3 * 64 + 16 * g + 4 * w;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t most = 0;
        Word4 part[3];
#pragma unroll
        for (int q = 0; q < 8; q += 2) {
            const float x0 = CT ? y[q / 4 * 4 + j][q % 4] : y[q][j], x1 = CT ? y[q / 4 * 4 + j][q % 4 + 1] : y[q + 1][j];
            most = max(most, max(__float_as_uint(x0) & 0x7fffffffu, __float_as_uint(x1) & 0x7fffffffu));
            split_pair(part, q / 2, x0, x1);
        }
        atomicMax(&cmax[16 * nbt + 4 * w + j], most);
#pragma unroll
        for (int i = 0; i < 3; ++i) to[64 * i + j] = part[i];
    }
}

// C as it is in the place of its parts (split_whole), all of it by one workgroup.
template <int KS2, int NBC>
__device__ __forceinline__ void write_whole(Word4 *Cl, const SplitC &c, bool transposed, int blocks) {
#pragma unroll 1
    for (int i = threadIdx.x; i < blocks * KS2 * 128; i += (int)blockDim.x) {
        const int l = i & 63, half = i >> 6 & 1, s = (i >> 7) % KS2, nbt = (i >> 7) / KS2;
        const int col = min(16 * nbt + (l & 12), c.cols - 4) + (l & 3), k0 = 32 * s + 16 * half + 4 * (l >> 4);
        auto number = [&](int k) __attribute__((always_inline)) {
            return k >= c.bcol ? 0u : __float_as_uint(c.C[transposed ? (int64_t)col * c.bcol + k : (int64_t)k * c.ld + col]);
        };
        Cl[(((nbt / NBC * KS2 + s) * NBC + nbt % NBC) * 3 + half) * 64 + l] = Word4{number(k0), number(k0 + 1), number(k0 + 2), number(k0 + 3)};
    }
}

// What a pass gathers: N entries of R rows, P pieces each.
template <typename Vec, int N, int R, int P> struct GatheredPieces {
    Vec v[N][R][P];
};

// KS: 16-byte pieces per lane of a row of B (bCol <= 4 V KS), NBC: blocks of sixteen columns of D
// multiplied at a time.
//
// A block's entries are gathered in passes of up to EM entries per row, with as many gathers on their way as the
// registers hold.  A wave adds up all passes of a block, multiplies, stores, and only then sends out the next block's
// first gathers: the other waves of its SIMD are at another step meanwhile, and the entries of a row are gathered at
// one time, so that what one wave fetches another finds in the L2 (2D stencil 512^2, fp64 128 -> 128: 373 MB fetched
// past the L2 and the matrix cores busy 62 % of the time; with the first pass on its way during the multiplications 657 MB,
// 190 us, so 182).  EARLY (chain_early): the first pass of the next block is sent out before the multiplications all the same.
//
// fp32 from depth 4 on, more than sixteen columns, is multiplied on the bf16 matrix cores, operands split in three (tf_device.h;
// chain_splits).
// These leave the other waves of their SIMD to work; behind fp32 and fp64 matrix instructions every instruction of
// theirs waits (loads, LDS reads or sums of four waves beside four that multiply take the sum of both times, beside
// bf16 instructions little more than the longer one).  us, before / with first gathers later and a piece of all entries
// in turn / on the bf16 matrix cores: 2D stencil 512^2, 64 -> 64 42 / 40 / 34.5, 128 -> 128 108 / 108 / 89; band of 15204
// rows of 41, 64 -> 64 15.8 / 14.0 / 12.5; 3D stencil 48^3, 64 -> 128 34.4 / 35.2 / 28.5.  Rows of B that are summed up
// outside of the bound of the split take the fp32 instructions, and all do if a column of C is, which sits in LDS as it is then
// (2D stencil 512^2, 128 -> 128: within 70, one column outside 104, every row 128; on the fp32 matrix cores alone 105).
template <typename T, int KS, int NBC, bool EARLY>
__global__ __launch_bounds__(kChainThreads, chain_waves(dtype_of<T>(), KS, NBC)) void k_gather_gemm(
    const ChainLaunch a, const ChainBlock *__restrict__ blocks, const int32_t *__restrict__ rows,
    const int32_t *__restrict__ idx, const T *__restrict__ val, const char *__restrict__ B,
    void *D) {
    constexpr int V = Tr<T>::V, KC = 4 * V;
    constexpr int EM = chain_entries(dtype_of<T>(), KS, EARLY);
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
    constexpr bool SPLIT = chain_splits(dtype_of<T>(), KS, NBC);     // (fp32 on the bf16 matrix cores)
    constexpr int KS2 = (KS + 1) / 2;
    T *Cl = reinterpret_cast<T *>(tf_smem);
    // the column groups of this workgroup (all of them, unless the launch has few blocks of rows)
    const int g0 = (int)blockIdx.y * a.groups_per_wg;
    const int groups = min(a.groups_per_wg, a.n_groups - g0), col0 = g0 * NBC * 16;
    // behind C, per wave: the place where pieces change lanes -- sums into operands (TS x 16 rows x 64
    // bytes; the pieces of a row are swizzled so that the sixteen rows' pieces g sit in different
    // banks), results into rows of D (16 rows of CB blocks and 16 bytes) -- then the offsets of the
    // rows of D and the entries of a pass (ES values, then addresses of rows of B)
    constexpr int ES = chain_entry_slots(dtype_of<T>(), KS, EARLY);
    constexpr int NE = chain_entry_loads(dtype_of<T>(), KS, EARLY), TS = chain_exchange(KS), CB = chain_store_blocks(dtype_of<T>(), KS, NBC);
    constexpr int W = CB * 16 / V, PITCH = W * 16 + 16;
    unsigned char *ex = tf_smem + a.groups_per_wg * (int)chain_group_lds(dtype_of<T>(), KS, NBC) +
                        wave * (int)chain_wave_lds(dtype_of<T>(), KS, NBC, EARLY);
    uint32_t *er = reinterpret_cast<uint32_t *>(ex + chain_exchange_bytes(dtype_of<T>(), KS, NBC));
    T *ev = reinterpret_cast<T *>(er + 16);
    uint64_t *ea = reinterpret_cast<uint64_t *>(ev + ES);
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
            if (ES >= e * 64 + 64 || lane < ES - e * 64) ea[e * 64 + lane] = at ^ ((at ^ zeros) & (uint64_t)(int64_t)pad);
        }
#pragma unroll
        for (int e = 0; e < NE; ++e)
            if (ES >= e * 64 + 64 || lane < ES - e * 64) ev[e * 64 + lane] = vi[e];
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

    T acc[RS][KP][V];
    // One pass: the gathers of n entries per row (known to the compiler), a piece of all entries in turn (neighbouring entries
    // name neighbouring rows of B, of which the piece before has fetched most: 2D stencil, fp32 64 -> 64, 39.2 -> 36.4 us), and
    // their sum.
    auto gather = [&](auto n_c, auto &x) __attribute__((always_inline)) {
        constexpr int N = decltype(n_c)::value;
        GlobalBytes p[N][RS];
#pragma unroll
        for (int e = 0; e < N; ++e)
#pragma unroll
            for (int h = 0; h < RS; ++h) p[e][h] = (GlobalBytes)(ea[e * 16 + rr + h * (64 / LR)] + first);
#pragma unroll
        for (int h = 0; h < RS; ++h)
#pragma unroll
            for (int t = 0; t < KP; ++t)
#pragma unroll
                for (int e = 0; e < N; ++e)
                    x.v[e][h][t] = *(GlobalVec)(t < T0 ? p[e][h] + 16 * LR * t : p[e][h] + moved[t < T0 ? 0 : t - T0]);
    };
    auto add_up = [&](auto n_c, const auto &x) __attribute__((always_inline)) {
        constexpr int N = decltype(n_c)::value;
        // All values first: one trip to LDS and back (band of 15204 rows of 41, fp32 19 -> 16, 9.76 -> 8.95 us).
        T w[N][RS];
#pragma unroll
        for (int e = 0; e < N; ++e)
#pragma unroll
            for (int h = 0; h < RS; ++h) w[e][h] = ev[e * 16 + rr + h * (64 / LR)];
#pragma unroll
        for (int e = 0; e < N; ++e)
#pragma unroll
            for (int h = 0; h < RS; ++h) asm volatile("" : "+v"(w[e][h]));
#pragma unroll
        for (int h = 0; h < RS; ++h)
#pragma unroll
            for (int t = 0; t < KP; ++t)
#pragma unroll
                for (int e = 0; e < N; ++e)
#pragma unroll
                    for (int q = 0; q < V; ++q) acc[h][t][q] += w[e][h] * x.v[e][h][t][q];
        __builtin_amdgcn_wave_barrier();
    };
    // calls f(n) with the count (1 to EM, wave-uniform) as a constant
    auto with_count = [&](int n, auto &&f) __attribute__((always_inline)) {
        auto from = [&](auto &self, auto n_c) __attribute__((always_inline)) -> void {
            constexpr int N = decltype(n_c)::value;
            if (N == 1 || n >= N) f(n_c);
            else if constexpr (N > 1) self(self, std::integral_constant<int, N - 1>());
        };
        from(from, std::integral_constant<int, EM>());
    };
    // A pass whose sums are formed later: n entries per row (wave-uniform: a branch per entry).
    auto send_first = [&](int n, GatheredPieces<Vec, EM, RS, KP> &x) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < EM; ++e) {
            if (e >= n) continue;
#pragma unroll
            for (int h = 0; h < RS; ++h) {
                const GlobalBytes p = (GlobalBytes)(ea[e * 16 + rr + h * (64 / LR)] + first);
#pragma unroll
                for (int t = 0; t < KP; ++t)
                    x.v[e][h][t] = *(GlobalVec)(t < T0 ? p + 16 * LR * t : p + moved[t < T0 ? 0 : t - T0]);
            }
        }
    };
    auto add_first = [&](int n, const GatheredPieces<Vec, EM, RS, KP> &x) __attribute__((always_inline)) {
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
            if (e >= n) continue;
#pragma unroll
            for (int h = 0; h < RS; ++h)
#pragma unroll
                for (int t = 0; t < KP; ++t)
#pragma unroll
                    for (int q = 0; q < V; ++q) acc[h][t][q] += w[e][h] * x.v[e][h][t][q];
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto clear_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < RS; ++h)
#pragma unroll
            for (int t = 0; t < KP; ++t)
#pragma unroll
                for (int q = 0; q < V; ++q) acc[h][t][q] = T(0);
    };
    auto pass_len = [](const ChainBlock &b) { return (b.info >> 3) & 15; };
    auto first_count = [&](const ChainBlock &b) { return min(pass_len(b), b.slots); };

    uint32_t *cmax = reinterpret_cast<uint32_t *>(tf_smem + groups * (NBC * KS2 * 3 * 1024));
    bool c_bad = false;      // (fp32) a column of C is outside of the bound of the split,
    float row_bound = 0.0f;  // what the elements of a row must be below
    GatheredPieces<Vec, EM, RS, KP> ahead;      // the first pass of the first block; EARLY: all passes
    // Start-up: the first gathers of the first block go out before C is put into LDS
    {
        const int total = groups * NBC * 16 * KS * 4, split_items = groups * NBC * KS2 * 16;
        const SplitC split_from{static_cast<const float *>(a.C) + (a.c_transposed ? (int64_t)col0 * a.bcol : col0), a.ccol, a.bcol, a.ccol - col0};
        CPiece<T> tmp[kStageC];
        const int n = blk < end ? first_count(d) : 0;
        auto first_gathers = [&]() __attribute__((always_inline)) {
            if (blk >= end) return;
            put();
            fetch(d.slots > pass_len(d) ? d.slot_base + pass_len(d) : dn.slot_base);
            send_first(n, ahead);
        };
        auto stage = [&](auto ct_c) __attribute__((always_inline)) {
            constexpr bool CT = decltype(ct_c)::value;
            load_c<T, KS, NBC, CT>(tmp, threadIdx.x, total, groups, col0, a);
            first_gathers();
            write_c<T, NBC, CT>(Cl, tmp);
            for (int p0 = (int)threadIdx.x + kStageC * (int)blockDim.x; p0 < total;
                 p0 += kStageC * (int)blockDim.x) {
                load_c<T, KS, NBC, CT>(tmp, p0, total, groups, col0, a);
                write_c<T, NBC, CT>(Cl, tmp);
            }
        };
        if constexpr (SPLIT) {
            auto stage_split = [&](auto ct_c) __attribute__((always_inline)) {
                constexpr bool CT = decltype(ct_c)::value;
                const int items = split_items;
                const SplitC &from = split_from;
                Word4 *const to = reinterpret_cast<Word4 *>(Cl);
                floatx4 y[8];
                load_split<KS2, CT>(y, from, threadIdx.x, items);
                for (int i = threadIdx.x; i < groups * NBC * 16; i += (int)blockDim.x) cmax[i] = 0;
                __syncthreads();
                first_gathers();
                write_split<KS2, NBC, CT>(to, cmax, y, threadIdx.x, items);
                for (int p = (int)threadIdx.x + (int)blockDim.x; p < items; p += (int)blockDim.x) {
                    load_split<KS2, CT>(y, from, p, items);
                    write_split<KS2, NBC, CT>(to, cmax, y, p, items);
                }
            };
            if (a.c_transposed) stage_split(std::true_type());
            else stage_split(std::false_type());
        } else {
            if (a.c_transposed) stage(std::true_type());
            else stage(std::false_type());
        }
        __syncthreads();
        if constexpr (!SPLIT)
            if (blk >= end) return;
        __builtin_amdgcn_s_waitcnt(0);
        asm volatile("" : : "v"(zeros_ahead));
        clear_sums();
        if constexpr (!EARLY) add_first(n, ahead);
        if constexpr (SPLIT) {
            row_bound = split_row_bound(cmax, groups * NBC * 16, lane, c_bad);
            if (c_bad) {      // (all waves of the workgroup; C as it is in the place of its parts)
                write_whole<KS2, NBC>(reinterpret_cast<Word4 *>(Cl), split_from, a.c_transposed, groups * NBC);
                __syncthreads();
            }
            if (blk >= end) return;
        }
    }

    for (int s0 = pass_len(d);; s0 = EARLY ? pass_len(d) : 0) {
        const int next = block_after(blk);
        const bool has_next = next < end;
        const ChainBlock dnn = blocks[min(block_after(next), end - 1)];
        if constexpr (EARLY) {
            clear_sums();
            add_first(first_count(d), ahead);
        }
        for (const int len = pass_len(d); s0 < d.slots; s0 += len) {
            if (s0) {
                put();
                fetch(s0 + len < d.slots ? d.slot_base + s0 + len : dn.slot_base);
            }
            const int count = min(len, d.slots - s0);
            if constexpr (EARLY) {
                send_first(count, ahead);
                add_first(count, ahead);
            } else {
                with_count(count, [&](auto n_c) __attribute__((always_inline)) {
                    GatheredPieces<Vec, decltype(n_c)::value, RS, KP> x;
                    gather(n_c, x);
                    add_up(n_c, x);
                });
            }
        }
        // the entries of the next block's first pass (the last block's wave takes those of some block, for nothing)
        put();
        row_n = row_id(dn);
        fetch(dn.slots > pass_len(dn) ? dn.slot_base + pass_len(dn) : dnn.slot_base);
        if constexpr (EARLY) send_first(first_count(dn), ahead);
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
        // wait for what was sent out before (the next pass's entries, EARLY the next block's gathers) does not
        // include them.  Gathers that follow the stores do wait for these, while other waves of the SIMD go on.  (us, with a
        // branch / without: 2D stencil 512^2, fp32 64 -> 64 32.2 / 31.6, 16 -> 16 9.40 / 9.29, fp64 128 -> 128 188.8 / 187.1, 32 -> 32
        // 27.8 / 28.4, band of 20011 rows, fp32 64 -> 64, 8.93 / 8.78.)
        if (g == 0)
            er[r] = (r >> slog) < n_rows && (r & ((1 << slog) - 1)) == 0 ? (uint32_t)row * (uint32_t)a.ccol : ~0u;
        const bool empty = d.slots == 0;      // (empty rows are zeros whatever C holds)
        __builtin_amdgcn_s_setprio(0);
        typedef typename Tr<T>::Acc Acc;
        auto each_group = [&](auto multiply) __attribute__((always_inline)) {
            int grp = 0;
            do {
                Acc o[NBC];
#pragma unroll
                for (int nb = 0; nb < NBC; ++nb) o[nb] = Acc{0, 0, 0, 0};
                multiply(grp, o);
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
        };
        if constexpr (!SPLIT) {
            each_group([&](int grp, Acc(&o)[NBC]) __attribute__((always_inline)) {
                // (the operands of a step are read ahead of the multiplications of the one before: 2D stencil 301^2, fp32 50 ->
                // 23, on the fp32 matrix cores 12.8 -> 12.3 us; further ahead where a step has few of them)
                constexpr int AHEAD = NBC == 1 ? 4 : NBC == 2 ? 2 : EARLY ? 0 : 1;
                const T *Cg = Cl + grp * (NBC * KS * V * 64) + lane;
                T c[AHEAD + 1][NBC];
#pragma unroll
                for (int i = 0; i < AHEAD && i < KS * V; ++i)
#pragma unroll
                    for (int nb = 0; nb < NBC; ++nb) c[i][nb] = Cg[(i * NBC + nb) * 64];
#pragma unroll
                for (int i = 0; i < KS * V; ++i) {
                    if (i + AHEAD < KS * V) {
#pragma unroll
                        for (int nb = 0; nb < NBC; ++nb) c[(i + AHEAD) % (AHEAD + 1)][nb] = Cg[((i + AHEAD) * NBC + nb) * 64];
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int nb = 0; nb < NBC; ++nb) o[nb] = mfma16(c[i % (AHEAD + 1)][nb], f[i / V][i % V], o[nb]);
                }
            });
        } else if constexpr (SPLIT) {
            float most = 0.0f;
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int q = 0; q < V; q += 2) most = fmaxf(fmaxf(most, fabsf(f[s][q])), fabsf(f[s][q + 1]));
            most = fmaxf(most, __shfl_xor(most, 16, 64));
            most = fmaxf(most, __shfl_xor(most, 32, 64));
            if (__builtin_amdgcn_ballot_w64(c_bad || split_exceeds(most, row_bound))) {
                each_group([&](int grp, Acc(&o)[NBC]) __attribute__((always_inline)) {
                    const Word4 *Cg = reinterpret_cast<const Word4 *>(Cl) + grp * (NBC * KS2 * 3 * 64) + lane;
#pragma unroll
                    for (int s = 0; s < KS2; ++s)
#pragma unroll
                        for (int nb = 0; nb < NBC; ++nb) {
                            float c[8];
                            split_whole(c, Cg + (s * NBC + nb) * 3 * 64, c_bad);
#pragma unroll
                            for (int q = 0; q < 8; ++q)
                                if (2 * s + q / 4 < KS) o[nb] = mfma16(c[q], f[2 * s + q / 4 < KS ? 2 * s + q / 4 : 0][q % 4], o[nb]);
                        }
                });
            } else {
                Word4 part[KS2][3];
                each_group([&](int grp, Acc(&o)[NBC]) __attribute__((always_inline)) {
                    const Word4 *Cg = reinterpret_cast<const Word4 *>(Cl) + grp * (NBC * KS2 * 3 * 64) + lane;
                    Acc small[NBC] = {};
#pragma unroll
                    for (int s = 0; s < KS2; ++s) {
                        if (grp == 0) {
#pragma unroll
                            for (int h = 0; h < 2; ++h)
#pragma unroll
                                for (int q = 0; q < V; q += 2) {
                                    const int k = 2 * s + h;
                                    split_pair(part[s], 2 * h + q / 2, k < KS ? f[k < KS ? k : 0][q] : 0.0f, k < KS ? f[k < KS ? k : 0][q + 1] : 0.0f);
                                }
                        }
#pragma unroll
                        for (int nb = 0; nb < NBC; ++nb) {
                            const Word4 *at = Cg + (s * NBC + nb) * 3 * 64;
                            const Word4 c[3] = {at[0], at[64], at[128]};
                            small[nb] = mfma16_bf16(c[2], part[s][1], small[nb]);
                            o[nb] = mfma16_bf16(c[0], part[s][0], o[nb]);
                            small[nb] = mfma16_bf16(c[1], part[s][2], small[nb]);
                            small[nb] = mfma16_bf16(c[2], part[s][0], small[nb]);
                            small[nb] = mfma16_bf16(c[0], part[s][2], small[nb]);
                            small[nb] = mfma16_bf16(c[1], part[s][1], small[nb]);
                            small[nb] = mfma16_bf16(c[1], part[s][0], small[nb]);
                            small[nb] = mfma16_bf16(c[0], part[s][1], small[nb]);
                        }
                    }
#pragma unroll
                    for (int nb = 0; nb < NBC; ++nb) o[nb] = split_sum(o[nb], small[nb]);
                });
            }
        }
        __builtin_amdgcn_s_setprio(3);
        if (!has_next) break;
        if constexpr (!EARLY) clear_sums();
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

template <typename T, int KS, int NBC, bool EARLY> int run_chain(ChainLaunch a, hipStream_t st) {
    static ChainSetup cs;
    auto kernel = k_gather_gemm<T, KS, NBC, EARLY>;
    // A launch with few blocks of rows is spread over the machine by column groups too (the rows are then
    // gathered once per group, and a workgroup stages its part of C only): as far as the machine holds all
    // its waves at once, half of them where C is small and little is saved (us, all groups in one workgroup /
    // as chosen: bands of 17 entries, fp64 128 -> 128, n = 4096 34.3 / 21.4, 8192 40.7 / 27.5, 16384 40.9 /
    // 32.1; fp32 128 -> 128 20.1 / 11.8, 23.7 / 13.3, 23.8 / 18.9; with twice the waves 51.5 at n = 16384 in fp64,
    // 34.7 / 24.0 at 32768 in fp32; C of 32 KiB, fp64 32 -> 128, n = 16384, 12.0 / 11.1 with one group each).
    // (by the size of C, whatever it takes in LDS)
    const int64_t group_bytes = (int64_t)NBC * KS * Tr<T>::V * 64 * (int64_t)sizeof(T);
    const int64_t group_lds = chain_group_lds(dtype_of<T>(), KS, NBC), wave_lds = chain_wave_lds(dtype_of<T>(), KS, NBC, EARLY);
    const int64_t held = (int64_t)a.n_cu * (a.n_groups * group_bytes <= 40 * 1024 ? 4 : 8);
    a.groups_per_wg = 1;
    while (a.n_blocks >= 2 * a.n_cu && a.groups_per_wg < a.n_groups &&
           (int64_t)a.n_blocks * ((a.n_groups + a.groups_per_wg - 1) / a.groups_per_wg) > held)
        ++a.groups_per_wg;
    // C in three parts may be more than the LDS holds, where C itself is not: then several workgroups take equal parts of the
    // column groups
    int n_y = (a.n_groups + a.groups_per_wg - 1) / a.groups_per_wg;
    while (a.groups_per_wg > 1 && a.groups_per_wg * group_lds + kChainThreads / 64 * wave_lds > a.lds_limit) {
        ++n_y;
        a.groups_per_wg = (a.n_groups + n_y - 1) / n_y;
    }
    n_y = (a.n_groups + a.groups_per_wg - 1) / a.groups_per_wg;
    const int64_t lds_c = a.groups_per_wg * group_bytes;
    // Waves per workgroup: one copy of C per workgroup, so the more LDS it takes the more waves have
    // to share it; a launch with fewer blocks than the machine has room for is spread thin, as far
    // as a wave does not have to stage more than 8 KiB of C.
    int waves = lds_c <= 40 * 1024 ? 4 : 8;
    while (waves > 1 && (int64_t)a.n_blocks * n_y < (int64_t)a.n_cu * waves && waves * 4096 >= lds_c) waves /= 2;
    const int64_t lds = a.groups_per_wg * group_lds + waves * wave_lds;
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

template <typename T, int KS, bool EARLY = false> int run_chain_nb(ChainLaunch a, hipStream_t st) {
    const int nb = (a.ccol + 15) / 16, nbc = chain_col_blocks(KS, a.ccol);
    a.n_groups = (nb + nbc - 1) / nbc;
    switch (nbc) {
        case 1: return run_chain<T, KS, 1, EARLY>(a, st);
        case 2: return run_chain<T, KS, 2, EARLY>(a, st);
    }
    if constexpr (KS < 16) return nbc == 3 ? run_chain<T, KS, 3, EARLY>(a, st) : run_chain<T, KS, 4, EARLY>(a, st);
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
            case 8: return a.early ? run_chain_nb<double, 8, true>(a, st) : run_chain_nb<double, 8>(a, st);
            case 12: return run_chain_nb<double, 12>(a, st);
            case 16: return run_chain_nb<double, 16>(a, st);
        }
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace tf
