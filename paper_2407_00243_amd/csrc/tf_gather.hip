// The kernels that gather rows: Y = A X over a packed list of rows of A (RowPack; the second wavefront, the second
// operation of the unfused baseline and of the plain pair, and Y = A B of the gather-first order), and Y = S X for a
// caller-supplied CSR matrix S.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "tf_device.h"

namespace tf {
namespace {

// What the kernels below are given beside the arrays that they read.  Small matrices wait for the host, whose time for a launch
// grows with the number and the bytes of its arguments; among them are 256 of the grid's sizes where a kernel asks for these, so the
// workgroups per XCD are handed over (the pair of launches, arguments of 504 and 440 bytes, 20 in all: 7.7 us of the host's
// time per call in some processes, 9.4 in others; 128 and 104, 15 in all: 7.5 and 8.7, and as `launch` does it now: below).
struct PackedArgs {
    void *Y, *partial;
    uint32_t *arrived;
    int64_t x_slice_stride;
    int32_t n_xs, sw, ldx, n_blocks, n_cut_blocks, ccol, contiguous, read_next, n_wg;
};
struct CsrArgs {
    void *Y, *D;
    int64_t y_slice_stride;
    int32_t n_rows, n_xs, x_sw, ccol, y_sw_shift, y_sw_mask, y_sw, n_wg;
};

// X is the D1 workspace (n_xs column slices of sw columns; idx is a slot) or a dense B (one slice).
//
// A wave owns a block of 64 / G virtual rows at a time (a row, or one of the 2^k parts that the rows of the
// block are cut into), G neighbouring lanes each; a lane holds 16 bytes of its row's columns.  The block's
// entries are gathered in passes of E per row: fetched a pass ahead with one coalesced load per 64 of them,
// turned into byte offsets of rows of X on the way to LDS (once per entry, not once per lane), read back
// from there by the lanes of their row.  Workgroups stay for all blocks of their share, four at a time, one
// for each wave; no barrier is passed, and the first gathers of the next block are on their way before a
// block's sums are stored.
//
// Slices: every XCD takes n_xs eighths of the blocks, of at most two slices, one after the other; an XCD's L2
// then holds sw-wide pieces of the hot rows instead of whole rows, and the eight caches hold different data.
// Blocks in the order of the rows (contiguous): an eighth is a range of blocks, through which the XCD's
// workgroups move side by side; blocks sorted by their slots are dealt back and forth, longest first.
//
// A row too long for one block takes the four blocks of a workgroup, whose waves add up their sums through LDS
// (the blocks of such rows come first), or several times that: these sums go past the L2 (device-scope stores
// and loads) and are there before the count of finished pieces is raised; the workgroup that is done last adds
// them up, in an order that does not depend on theirs.  The count goes round: every launch raises it by as many as
// there are pieces, so that it is back at zero after any number of launches, whatever they ran beside.
//
// Bound by the fabric behind the L2 where rows reach far: R-MAT graph of 2^20 vertices, fp32, 128 columns in four
// slices, 689 us, 4.8 GB cross the memory interface at 7.0 TB/s (units staged by a workgroup behind a barrier: 747
// us, 6.8 TB/s); 32 columns 178 us, 6.5 TB/s (205 us).  By the chain of loads where they do not: hence a pass of eight
// entries and the next one's offsets in flight at any time.
template <typename T, int VV, int G, bool WIDE>
__global__ __launch_bounds__(kSpmmThreads, gather_waves(dtype_of<T>())) void k_packed_spmm(
    const PackedArgs a, const GatherBlock *__restrict__ blocks, const int32_t *__restrict__ rows,
    const int32_t *__restrict__ lens, const int32_t *__restrict__ idx, const T *__restrict__ val,
    const CutBlock *__restrict__ cuts, const T *__restrict__ X0) {
    T *const Y0 = static_cast<T *>(a.Y), *const partial = static_cast<T *>(a.partial);
    uint32_t *const all_arrived = a.arrived;
    constexpr int E = kGatherEntries, NR = 64 / G, NE = NR * E > 64 ? NR * E / 64 : 1;
    typedef std::conditional_t<WIDE, uint64_t, uint32_t> Off;
    typedef T Vec16 __attribute__((ext_vector_type(Tr<T>::V)));
    typedef std::conditional_t<VV == 1, T, Vec16> X16;                          // a lane's columns of a row,
    typedef std::conditional_t<VV == 1, T, typename Piece16<T>::Vec> XAny;      // in device memory
    auto part = [](const X16 &x, int i) __attribute__((always_inline)) {
        if constexpr (VV == 1) return x;
        else return x[i];
    };
    __shared__ __align__(16) Off off_s[kSpmmThreads / 64][NR * E];
    __shared__ __align__(16) T val_s[kSpmmThreads / 64][NR * E];
    __shared__ __align__(16) T sum_s[kSpmmThreads / 64][G * VV];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int gl = lane % G, v = lane / G;
    Off *off_w = off_s[wave];
    T *val_w = val_s[wave];
    const Off row_bytes = (Off)a.ldx * (Off)sizeof(T);
    // (quads: the blocks of a workgroup)
    const int n_wg = a.n_wg, my = (int)(blockIdx.x / kXcds);
    const int n_quads = (uint32_t)a.n_blocks / kGatherQuad, eighth = (uint32_t)(n_quads + kXcds - 1) / kXcds;
    const int n_cb = (uint32_t)(a.sw + G * VV - 1) / (G * VV);        // column blocks of a slice (rows wider than a wave's load)

    int32_t ci[NE];
    T vi[NE];
    auto fetch = [&](uint32_t slot) __attribute__((always_inline)) {
        const int64_t at = (int64_t)slot * NR + (lane & (NR * E - 1));
#pragma unroll
        for (int k = 0; k < NE; ++k) ci[k] = idx[at + 64 * k];
#pragma unroll
        for (int k = 0; k < NE; ++k) vi[k] = val[at + 64 * k];
    };
    auto put = [&]() __attribute__((always_inline)) {
        if (NR * E >= 64 || lane < NR * E) {
#pragma unroll
            for (int k = 0; k < NE; ++k) {
                const int l = lane + 64 * k, to = l % NR * E + l / NR;
                off_w[to] = (Off)(uint32_t)ci[k] * row_bytes;
                val_w[to] = vi[k];
            }
        }
        __builtin_amdgcn_wave_barrier();
    };

    // (n_xs > 0: a loop that ends with its test, or the arguments are fetched in two rounds)
    int at = (int)(blockIdx.x % kXcds) * a.n_xs, left = a.n_xs;
    do {
        const int slice = at / kXcds, e0 = at % kXcds, n_e = min(left, kXcds - e0);
        at += n_e;
        left -= n_e;
        const int w = min(a.sw, a.ccol - slice * a.sw);     // columns of this slice
        uint32_t reciprocal = 0;                            // 2^32 / n_e, rounded up
#pragma unroll
        for (int k = 2; k <= kXcds; ++k) reciprocal = n_e == k ? 0xffffffffu / k + 1 : reciprocal;
        // quad of the workgroup's k-th round: the XCD's quads in their order, or dealt back and forth
        const int end = a.contiguous ? min(n_quads, (e0 + n_e) * eighth) : n_quads;
        auto quad_of = [&](int k) __attribute__((always_inline)) {
            if (a.contiguous) return e0 * eighth + k * n_wg + my;
            const int j = k * n_wg + (k & 1 ? n_wg - 1 - my : my);
            const int q = n_e == 1 ? j : (int)__umulhi((uint32_t)j, reciprocal);       // j / n_e
            return q * kXcds + e0 + j - q * n_e;
        };
        int cb = 0;
        do {
            const bool active = cb * G * VV + VV * gl < w;
            const int col = min(cb * G * VV + VV * gl, w - VV);
            const char *__restrict__ X = reinterpret_cast<const char *>(X0 + (int64_t)slice * a.x_slice_stride);
            const Off lane_bytes = (Off)col * (Off)sizeof(T);
            T *Yl = Y0 + slice * a.sw + col;

            X16 x[E];
            T acc[VV];
            auto issue = [&](int n) __attribute__((always_inline)) {
                Off o[E];
#pragma unroll
                for (int e = 0; e < E; e += 16 / (int)sizeof(Off))
                    load_pack<Off, 16 / (int)sizeof(Off)>(*reinterpret_cast<Off(*)[16 / sizeof(Off)]>(&o[e]), off_w + v * E + e);
                // (all offsets in one trip to LDS; what x held is dead: said so, or the compiler keeps it beside what is
                // loaded)
#pragma unroll
                for (int e = 0; e < E; ++e) asm volatile("" : "+v"(o[e]));
#pragma unroll
                for (int e = 0; e < E; ++e) asm volatile("" : "=v"(x[e]));
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (e < n) x[e] = *reinterpret_cast<const XAny *>(X + (Off)(o[e] + lane_bytes));
            };
            // whole: all virtual rows have the n entries of the pass; else n_real: those of the lane's row, and what lies
            // beyond adds nothing, whatever X holds
            auto consume = [&](int n, bool whole, int n_real) __attribute__((always_inline)) {
                T f[E];
#pragma unroll
                for (int e = 0; e < E; e += Tr<T>::V)
                    load_pack<T, Tr<T>::V>(*reinterpret_cast<T(*)[Tr<T>::V]>(&f[e]), val_w + v * E + e);
                if (whole) {
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        if (e < n) {
#pragma unroll
                            for (int i = 0; i < VV; ++i) acc[i] += f[e] * part(x[e], i);
                        }
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < E; ++e)
#pragma unroll
                        for (int i = 0; i < VV; ++i) acc[i] += (e < n_real ? f[e] : T(0)) * (e < n_real ? part(x[e], i) : T(0));
                }
                __builtin_amdgcn_wave_barrier();
            };
            auto slots = [](const GatherBlock &b) { return (int)(b.size & 0xffff); };
            auto row_at = [&](const GatherBlock &b) __attribute__((always_inline)) {
                const int each = (b.info >> 3) & 7;
                const int at = each ? v * gather_short_rows(each, G) + gl % gather_short_rows(each, G) : v >> (b.info & 7);
                return b.row_begin + max(0, min(at, (int)(b.info >> 6) - 1));
            };
            auto put_row = [&](int32_t row, const T(&v)[VV]) __attribute__((always_inline)) {
                XAny y;
                if constexpr (VV == 1) y = v[0];
                else
#pragma unroll
                    for (int i = 0; i < VV; ++i) y[i] = v[i];
                XAny *to = reinterpret_cast<XAny *>(Yl + (int64_t)row * a.ccol);
                // (a Y that is not read again soon passes through the L2: what it would evict there is)
                if (a.read_next) *to = y;
                else __builtin_nontemporal_store(y, to);
            };
            auto finish = [&](const GatherBlock &b, int32_t row, int at_block) __attribute__((always_inline)) {
                const int slog = (int)(b.info & 7);
                for (int m = G; m < G << slog; m <<= 1) {
#pragma unroll
                    for (int i = 0; i < VV; ++i) acc[i] += __shfl_xor(acc[i], m, 64);
                }
                bool store = active && (v & ((1 << slog) - 1)) == 0 && (v >> slog) < (int)(b.info >> 6);
                const bool cut = at_block < a.n_cut_blocks;      // (the same for all four blocks of the quad)
                if (cut) {
                    if (v == 0) store_pack<T, VV>(&sum_s[wave][gl * VV], acc);
                    __syncthreads();
                    if (wave == 0) {
#pragma unroll
                        for (int i = 0; i < VV; ++i) acc[i] = T(0);
                        for (int k = 0; k < kGatherQuad; ++k)
#pragma unroll
                            for (int i = 0; i < VV; ++i) acc[i] += sum_s[k][gl * VV + i];
                    }
                    __syncthreads();
                    if (wave != 0) return;
                }
                if (cut && cuts[at_block].pieces > 1) {
                    const CutBlock c = cuts[at_block];
                    const int64_t pitch = (int64_t)a.n_xs * a.sw;
                    T *p = partial + slice * a.sw + col;
                    if (store) {
#pragma unroll
                        for (int i = 0; i < VV; ++i)
                            __hip_atomic_store(p + c.piece * pitch + i, acc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __builtin_amdgcn_s_waitcnt(0);
                    uint32_t *arrived = all_arrived + ((int64_t)c.row * a.n_xs + slice) * n_cb + cb;
                    const uint32_t last = (uint32_t)__builtin_amdgcn_readfirstlane(c.pieces) - 1;
                    uint32_t done = 0;
                    if (lane == 0) done = atomicInc(arrived, last);
                    if ((uint32_t)__builtin_amdgcn_readfirstlane(done) != last) return;
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
                    for (int i = 0; i < VV; ++i) acc[i] = T(0);
                    for (int k = v; k < c.pieces; k += NR) {
#pragma unroll
                        for (int i = 0; i < VV; ++i)
                            acc[i] += __hip_atomic_load(p + (c.first_piece + k) * pitch + i, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
                    }
                    for (int m = G; m < 64; m <<= 1) {
#pragma unroll
                        for (int i = 0; i < VV; ++i) acc[i] += __shfl_xor(acc[i], m, 64);
                    }
                }
                if (store) put_row(row, acc);
            };
            // rows of S entries, several to a lane group: the pass holds all of them
            auto finish_short = [&](auto each, const GatherBlock &b, int32_t row) __attribute__((always_inline)) {
                constexpr int S = decltype(each)::value, R = gather_short_rows(S, G);
                T f[E];
#pragma unroll
                for (int e = 0; e < E; e += Tr<T>::V)
                    load_pack<T, Tr<T>::V>(*reinterpret_cast<T(*)[Tr<T>::V]>(&f[e]), val_w + v * E + e);
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    T y[VV];
#pragma unroll
                    for (int i = 0; i < VV; ++i) y[i] = T(0);
#pragma unroll
                    for (int e = k * S; e < k * S + S; ++e)
#pragma unroll
                        for (int i = 0; i < VV; ++i) y[i] += f[e] * part(x[e], i);
                    const int32_t to = __shfl(row, v * G + k, 64);
                    if (active && v * R + k < (int)(b.info >> 6)) put_row(to, y);
                }
                __builtin_amdgcn_wave_barrier();
            };

            int k = 0, u = quad_of(k);
            if (u >= end) break;
            int at_d = u * kGatherQuad + wave, at_n = at_d;
            GatherBlock d = blocks[at_d], dn = d;
            int32_t row = rows[row_at(d)], len = lens[row_at(d)];
            fetch(d.slot_base);
            u = quad_of(++k);
            bool has_next = u < end;
            if (has_next) dn = blocks[at_n = u * kGatherQuad + wave];
            put();
            fetch(slots(d) > E ? d.slot_base + E : dn.slot_base);
            issue(min(E, slots(d)));
            for (;;) {
                u = quad_of(++k);
                const bool has_next2 = has_next && u < end;
                GatherBlock dnn = dn;
                int at_nn = at_n;
                if (has_next2) dnn = blocks[at_nn = u * kGatherQuad + wave];
#pragma unroll
                for (int i = 0; i < VV; ++i) acc[i] = T(0);
                // entries of the lane's (virtual) row
                const int n_d = slots(d), whole = (int)(d.size >> 16), skip = at_d < a.n_cut_blocks ? cuts[at_d].skip : 0;
                const int real = min(n_d, len - (v & ((1 << (d.info & 7)) - 1)) * n_d - skip);
                const int each = (d.info >> 3) & 7;
                if (each) {
                    if (G >= 8 && each == 1) finish_short(std::integral_constant<int, 1>(), d, row);
                    else if (G >= 4 && each == 2) finish_short(std::integral_constant<int, 2>(), d, row);
                    else if (G >= 2 && each == 3) finish_short(std::integral_constant<int, 3>(), d, row);
                    else if (G >= 2) finish_short(std::integral_constant<int, 4>(), d, row);
                } else {
                    consume(min(E, n_d), whole >= min(E, n_d), real);
                }
                for (int s0 = E; s0 < n_d; s0 += E) {
                    put();
                    fetch(s0 + E < n_d ? d.slot_base + s0 + E : dn.slot_base);
                    issue(min(E, n_d - s0));
                    consume(min(E, n_d - s0), whole >= min(s0 + E, n_d), real - s0);
                }
                // the next block's first gathers go out before this one's sums are stored (none after the last)
                int32_t row_n = 0, len_n = 0;
                if (has_next) {
                    put();
                    row_n = rows[row_at(dn)];
                    len_n = lens[row_at(dn)];
                    fetch(slots(dn) > E ? dn.slot_base + E : dnn.slot_base);
                }
                issue(has_next ? min(E, slots(dn)) : 0);
                if (!each) finish(d, row, at_d);
                if (!has_next) break;
                d = dn;
                dn = dnn;
                at_d = at_n;
                at_n = at_nn;
                row = row_n;
                len = len_n;
                has_next = has_next2;
            }
        } while (++cb < n_cb && cb * G * VV < w);
    } while (left > 0);
}

// Y[j] = S[j, :] X for a caller-supplied CSR matrix S: the first operation of the unfused SpMM-SpMM baseline and of
// the plain pair (row_info = nullptr: every row goes to the workspace, slot = row), and the first wavefront of a
// CSR-B plan that needs no tile in LDS (row_info: what happens to a finished D1 row, see kInfo*; a row whose D1
// row nobody reads and that the plan leaves out counts as empty, nothing of it is fetched).
//
// As k_packed_spmm, for rows as they come: a wave owns 64 / G consecutive rows at a time and takes E entries of each
// per pass.  What the passes need of the rows' extents is read two blocks ahead, entries a pass ahead, the first
// gathers of the next block go out before a block's rows are stored.  Every XCD takes n_xs eighths of the rows, of
// at most two column slices of X.  The time of a block is that of its longest row; which wave takes which, CsrWalk.
// Bound as k_packed_spmm: 2^20 rows of eight random columns, fp32, 32 columns, 190 us, 5.7 TB/s of gathered lines (184
// us when workgroups staged entries behind barriers, 181 with two workgroups per compute unit: run_csr); 3000 rows of
// 49, 100 columns, both operations 13.8 us (44.4).  Rows of one or two lanes are fetched for by all lanes alike, eight
// entries a pass as the others (four, to have registers for 64 extents a lane: 30000 rows of a graph, fp32, 6 columns,
// both operations 382 us, now 321; the extents come from the rows' lanes once a block).
template <typename T, int VV, int G, int E, bool WIDE>
__global__ __launch_bounds__(kSpmmThreads, csr_waves(dtype_of<T>(), G)) void k_csr_spmm(
    const CsrArgs a, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const T *__restrict__ vals, const T *__restrict__ X0, const uint32_t *__restrict__ row_info,
    const T *__restrict__ row_scale) {
    T *const Y = static_cast<T *>(a.Y), *const D = static_cast<T *>(a.D);
    constexpr int NR = 64 / G, NE = NR * E > 64 ? NR * E / 64 : 1;
    typedef std::conditional_t<WIDE, uint64_t, uint32_t> Off;
    typedef T Vec16 __attribute__((ext_vector_type(Tr<T>::V)));
    typedef std::conditional_t<VV == 1, T, Vec16> X16;                          // a lane's columns of a row,
    typedef std::conditional_t<VV == 1, T, typename Piece16<T>::Vec> XAny;      // in device memory
    auto part = [](const X16 &x, int i) __attribute__((always_inline)) {
        if constexpr (VV == 1) return x;
        else return x[i];
    };
    __shared__ __align__(16) Off off_s[kSpmmThreads / 64][NR * E];
    __shared__ __align__(16) T val_s[kSpmmThreads / 64][NR * E];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int gl = lane % G, v = lane / G;
    Off *off_w = off_s[wave];
    T *val_w = val_s[wave];
    const Off row_bytes = (Off)a.ccol * (Off)sizeof(T);
    const CsrBlocks all{(uint32_t)a.n_rows, NR};
    const uint32_t n_waves = (uint32_t)a.n_wg * (kSpmmThreads / 64);
    const uint32_t my = blockIdx.x / kXcds * (kSpmmThreads / 64) + (uint32_t)wave;
    const int n_cb = (uint32_t)(a.x_sw + G * VV - 1) / (G * VV);

    // of a block: the extent of the row whose entries the lane fetches (where these are several rows, that of the one that
    // it sums up), and what becomes of the row that it sums up
    struct Rows {
        int32_t kb, ke, len;
        uint32_t info;
        T scale;
    };
    typedef int32_t Extent __attribute__((ext_vector_type(2), aligned(4)));
    auto read_rows = [&](uint32_t u) __attribute__((always_inline)) {
        Rows b;
        const uint32_t j = all.row(u, v), r = NE > 1 ? j : all.row(u, lane % (NR * E) / E);
        const Extent x = *reinterpret_cast<const Extent *>(rowptr + r);
        uint32_t info = row_info ? row_info[r] : 0u;
        b.kb = x[0];
        b.ke = info & kInfoSkip ? x[0] : x[1];
        b.len = b.ke - b.kb;
        if constexpr (NE == 1 && G != E) {
            // (the lane's row is that of a lane v E; with eight lanes a row, its own)
            b.len = __shfl(b.len, v * E, 64);
            info = __shfl(info, v * E, 64);
        }
        b.info = d1_info(row_info != nullptr, info);
        b.scale = row_scale ? row_scale[j] : T(0);
        if (!all.has(u, v)) {
            b.len = 0;
            b.info = 0;
        }
        return b;
    };
    int32_t ci[NE], fb[NE], fe[NE];
    T vi[NE];
    // the block whose entries are fetched from here on
    auto aim = [&](const Rows &b) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            fb[k] = b.kb;
            fe[k] = b.ke;
            if constexpr (NE > 1) {
                fb[k] = __shfl(b.kb, (lane + 64 * k) / E * G, 64);
                fe[k] = __shfl(b.ke, (lane + 64 * k) / E * G, 64);
            }
        }
    };
    auto fetch = [&](uint32_t s0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            const uint32_t s = s0 + lane % E;
            ci[k] = 0;
            vi[k] = T(0);
            if (has_entry(fb[k], fe[k], s)) {
                const int at = fb[k] + (int)s;
                ci[k] = colidx[at];
                vi[k] = vals[at];
            }
        }
    };
    auto put = [&]() __attribute__((always_inline)) {
        if (NR * E >= 64 || lane < NR * E) {
#pragma unroll
            for (int k = 0; k < NE; ++k) {
                off_w[lane + 64 * k] = (Off)(uint32_t)ci[k] * row_bytes;
                val_w[lane + 64 * k] = vi[k];
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto any = [](bool x) { return __builtin_amdgcn_ballot_w64(x) != 0; };

    int at = (int)(blockIdx.x % kXcds) * a.n_xs, left = a.n_xs;
    do {
        const int slice = at / kXcds, e0 = at % kXcds, n_e = min(left, kXcds - e0);
        at += n_e;
        left -= n_e;
        const int w = min(a.x_sw, a.ccol - slice * a.x_sw);     // columns of this slice
        const uint32_t end = all.end(e0 + n_e);
        int cb = 0;
        do {
            const bool active = cb * G * VV + VV * gl < w;
            const int col = slice * a.x_sw + min(cb * G * VV + VV * gl, w - VV);
            const char *__restrict__ X = reinterpret_cast<const char *>(X0);
            const Off lane_bytes = (Off)col * (Off)sizeof(T);
            // the lane's columns of a row of the workspace (slices of y_sw columns) and of D
            T *Yl = Y + (int64_t)(col >> a.y_sw_shift) * a.y_slice_stride + (col & a.y_sw_mask);
            T *Dl = D + col;
            X16 x[E];
            T acc[VV];
            // left: entries that the lane's row has from this pass on
            auto issue = [&](int rest) __attribute__((always_inline)) {
                Off o[E];
#pragma unroll
                for (int e = 0; e < E; e += 16 / (int)sizeof(Off))
                    load_pack<Off, 16 / (int)sizeof(Off)>(*reinterpret_cast<Off(*)[16 / sizeof(Off)]>(&o[e]), off_w + v * E + e);
#pragma unroll
                for (int e = 0; e < E; ++e) asm volatile("" : "+v"(o[e]));
#pragma unroll
                for (int e = 0; e < E; ++e) asm volatile("" : "=v"(x[e]));
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (any(e < rest)) x[e] = *reinterpret_cast<const XAny *>(X + (Off)(o[e] + lane_bytes));
            };
            auto consume = [&](int rest) __attribute__((always_inline)) {
                T f[E];
#pragma unroll
                for (int e = 0; e < E; e += Tr<T>::V)
                    load_pack<T, Tr<T>::V>(*reinterpret_cast<T(*)[Tr<T>::V]>(&f[e]), val_w + v * E + e);
                if (!any(rest < E)) {
#pragma unroll
                    for (int e = 0; e < E; ++e)
#pragma unroll
                        for (int i = 0; i < VV; ++i) acc[i] += f[e] * part(x[e], i);
                } else {
#pragma unroll
                    for (int e = 0; e < E; ++e)
#pragma unroll
                        for (int i = 0; i < VV; ++i) acc[i] += (e < rest ? f[e] : T(0)) * (e < rest ? part(x[e], i) : T(0));
                }
                __builtin_amdgcn_wave_barrier();
            };
            auto finish = [&](const Rows &b, uint32_t u) __attribute__((always_inline)) {
                if (!active) return;
                const int64_t j = u * NR + (uint32_t)v;
                if (b.info & kInfoSpill) store_any<T, VV>(Yl + d1_slot(row_info != nullptr, b.info, j) * a.y_sw, acc);
                if (b.info & (kInfoDirect | kInfoZero)) {
                    XAny y;
                    if constexpr (VV == 1) y = (b.info & kInfoZero) ? T(0) : b.scale * acc[0];
                    else
#pragma unroll
                        for (int i = 0; i < VV; ++i) y[i] = (b.info & kInfoZero) ? T(0) : b.scale * acc[i];
                    // (D is not read again: what it would evict from the L2 is)
                    __builtin_nontemporal_store(y, reinterpret_cast<XAny *>(Dl + j * a.ccol));
                }
            };

            CsrWalk u{e0 * all.eighth() + my, my};
            if (u.at >= end) break;
            CsrWalk un = u.next(n_waves);
            Rows d = read_rows(u.at), dn = read_rows(min(un.at, end - 1));
            // the entries of the pass behind: the block's next, or the first of the next block
            auto fetch_next = [&](bool more, uint32_t s, const Rows &next) __attribute__((always_inline)) {
                if (!more) aim(next);
                fetch(more ? s : 0);
            };
            aim(d);
            fetch(0);
            put();
            fetch_next(any(d.len > E), E, dn);
            issue(d.len);
            for (;;) {
                const bool has_next = un.at < end;
                const CsrWalk unn = un.next(n_waves);
                const Rows dnn = read_rows(min(unn.at, end - 1));
#pragma unroll
                for (int i = 0; i < VV; ++i) acc[i] = T(0);
                consume(d.len);
                for (uint32_t s0 = E; any(has_entry(0, d.len, s0)); s0 += E) {
                    put();
                    fetch_next(any(has_entry(0, d.len, s0 + E)), s0 + E, dn);
                    issue(d.len - (int)s0);
                    consume(d.len - (int)s0);
                }
                if (has_next) {
                    put();
                    fetch_next(any(dn.len > E), E, dnn);
                }
                issue(has_next ? dn.len : 0);      // (none after the last)
                finish(d, u.at);
                if (!has_next) break;
                d = dn;
                dn = dnn;
                u = un;
                un = unn;
            }
        } while (++cb < n_cb && cb * G * VV < w);
    } while (left > 0);
}

// A launch that returns its own status, in one call of the runtime; in chevrons, with the last error asked for before and after
// it, it is five (host time of a pair of launches of small matrices, 3 processes each, us: 9.0, 9.1, 9.0; now 8.4, 7.2, 7.2).
template <typename... P> int launch(void (*kernel)(P...), int64_t n_wg, hipStream_t st, std::decay_t<P>... args) {
    void *at[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3((unsigned)n_wg), dim3(kSpmmThreads), at, 0, st);
    if (e != hipSuccess) (void)hipGetLastError();      // (reported here, not by a later call)
    return (int)e;
}

template <typename T, int VV, int G, bool WIDE> int run_packed(const PackedSpmmLaunch &a, hipStream_t st) {
    // Where most rows come from beyond the L2, more requests on their way than two workgroups per compute unit have only
    // get in each other's way; where the L2 has them, they hide its latency (130 points, us, all / two: uniform columns, fp64
    // 36 columns, 700000 rows 342 / 313, 250000 119 / 110; R-MAT graph of 2^20, fp32, 90 columns 599 / 579; never slower below
    // half of the entries named again, up to 12 % slower at .58, 37 % at .7).
    static const int most = resident_per_cu(k_packed_spmm<T, VV, G, WIDE>, kSpmmThreads, 0, 8);
    const int wg_per_cu = a.few_waves ? std::min(most, 2) : most;
    const int64_t quads = ((int64_t)a.n_blocks / kGatherQuad + kXcds - 1) / kXcds * a.n_xs;        // of an XCD
    const int64_t per_xcd = std::min<int64_t>(quads, std::max(1, a.n_cu / kXcds) * (int64_t)wg_per_cu);
    PackedArgs k;
    k.Y = a.Y;
    k.partial = a.partial;
    k.arrived = a.arrived;
    k.x_slice_stride = a.x_slice_stride;
    k.n_xs = a.n_xs;
    k.sw = a.sw;
    k.ldx = a.ldx;
    k.n_blocks = a.n_blocks;
    k.n_cut_blocks = a.n_cut_blocks;
    k.ccol = a.ccol;
    k.contiguous = a.contiguous;
    k.read_next = a.read_next;
    k.n_wg = (int32_t)per_xcd;
    return launch(k_packed_spmm<T, VV, G, WIDE>, per_xcd * kXcds, st, k, a.pack.blocks, a.pack.rows, a.pack.lens, a.pack.idx,
                  static_cast<const T *>(a.pack.vals), a.pack.cuts, static_cast<const T *>(a.X));
}

template <typename T, int VV, int G, int E, bool WIDE> int run_csr(const CsrSpmmLaunch &a, hipStream_t st) {
    // (all that the machine holds: two per compute unit where X is beyond the caches and rows of S have six entries and
    // more are 0 to 5 % faster for random columns, but up to 65 % slower for columns near the diagonal, 85 % with long
    // rows among them, and S is not known before the call)
    static const int wg_per_cu = resident_per_cu(k_csr_spmm<T, VV, G, E, WIDE>, kSpmmThreads, 0, 8);
    const int64_t blocks = ((int64_t)a.n_rows + 64 / G - 1) / (64 / G), items = (blocks + kXcds - 1) / kXcds * a.n_xs;
    const int64_t per_xcd = std::min<int64_t>((items + kSpmmThreads / 64 - 1) / (kSpmmThreads / 64),
                                              std::max(1, a.n_cu / kXcds) * (int64_t)wg_per_cu);
    CsrArgs k;
    k.Y = a.Y;
    k.D = a.D;
    k.y_slice_stride = a.y_slice_stride;
    k.n_rows = a.n_rows;
    k.n_xs = a.n_xs;
    k.x_sw = a.x_sw;
    k.ccol = a.ccol;
    k.y_sw_shift = a.y_sw_shift;
    k.y_sw_mask = a.y_sw_mask;
    k.y_sw = a.y_sw;
    k.n_wg = (int32_t)per_xcd;
    return launch(k_csr_spmm<T, VV, G, E, WIDE>, per_xcd * kXcds, st, k, a.S.rowptr, a.S.colidx,
                  static_cast<const T *>(a.S.vals), static_cast<const T *>(a.X), a.row_info,
                  static_cast<const T *>(a.row_scale));
}

// Calls f(VV, G) with compile-time constants: columns and lanes of rows in column slices of sw of the ccol columns.
template <typename T, typename L> int dispatch_group(int64_t ccol, int sw, L &&f) {
    constexpr int V = Tr<T>::V;
    const int elems = lane_elems(dtype_of<T>(), ccol, sw), group = lane_group(sw, elems);
#define TF_G(VVV, GV) return f(std::integral_constant<int, VVV>(), std::integral_constant<int, GV>())
    if (elems == 1) {
        // (rows narrower than 16 bytes)
        switch (group) {
            case 1: TF_G(1, 1);
            case 2: TF_G(1, 2);
            case 4: TF_G(1, 4);
        }
        return (int)hipErrorInvalidValue;
    }
    switch (group) {
        case 1: TF_G(V, 1);
        case 2: TF_G(V, 2);
        case 4: TF_G(V, 4);
        case 8: TF_G(V, 8);
        case 16: TF_G(V, 16);
        case 32: TF_G(V, 32);
        case 64: TF_G(V, 64);
    }
#undef TF_G
    return (int)hipErrorInvalidValue;
}

template <typename T> int run_packed_group(const PackedSpmmLaunch &a, hipStream_t st) {
    return dispatch_group<T>(a.ccol, a.sw, [&](auto vv, auto g) {
        constexpr int VV = decltype(vv)::value, G = decltype(g)::value;
        return a.wide ? run_packed<T, VV, G, true>(a, st) : run_packed<T, VV, G, false>(a, st);
    });
}
template <typename T> int run_csr_group(const CsrSpmmLaunch &a, hipStream_t st) {
    return dispatch_group<T>(a.ccol, a.x_sw, [&](auto vv, auto g) {
        constexpr int VV = decltype(vv)::value, G = decltype(g)::value;
        // entries a pass: rows of one and two lanes, 64 and 32 in a wave, pay for passes that their entries do not fill
        // (30000 rows of three, fp32, 8 columns, both operations: four 6.35 us, eight 6.92; longer rows: k_csr_spmm)
        auto run = [&](auto e) {
            constexpr int E = decltype(e)::value;
            return a.x_bytes >= ((int64_t)1 << 32) ? run_csr<T, VV, G, E, true>(a, st) : run_csr<T, VV, G, E, false>(a, st);
        };
        if constexpr (G <= 2)
            if (a.mean_len <= 4) return run(std::integral_constant<int, 4>());
        return run(std::integral_constant<int, kGatherEntries>());
    });
}

}  // namespace

int launch_packed_spmm(const PackedSpmmLaunch &a, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (a.n_blocks == 0) return 0;
    if (a.n_xs < 1 || a.n_xs > kXcds || a.n_blocks % kGatherQuad) return (int)hipErrorInvalidValue;
    return a.dtype == TF_F32 ? run_packed_group<float>(a, st) : run_packed_group<double>(a, st);
}

int launch_csr_spmm(const CsrSpmmLaunch &a, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (a.n_rows == 0) return 0;
    if (a.n_xs < 1 || a.n_xs > kXcds) return (int)hipErrorInvalidValue;
    return a.dtype == TF_F32 ? run_csr_group<float>(a, st) : run_csr_group<double>(a, st);
}

}  // namespace tf
