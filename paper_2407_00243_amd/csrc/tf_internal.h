// Internal declarations shared by the inspector (host), the kernels (device) and the C ABI.
#pragma once
#include <cstdint>
#include <memory>
#include <new>
#include <utility>
#include <string>
#include <vector>

#include "../../include/tilefusion.h"

namespace tf {

// Limits of the kernels.
constexpr int kMaxMfmaSliceCols = 128;   // one wave holds at most 8 accumulator blocks of 16 columns
constexpr int kRowGranuleDense = 16;     // dense-B tiles are produced in blocks of 16 rows (MFMA M/N)
constexpr int kXcds = 8;                 // XCDs of the device: consecutive workgroup ids are dealt to them round robin,
                                         // each has its own L2 (the kernels' work-to-workgroup maps and the grid sizes use it)
constexpr int kFusedThreads = 512;       // workgroup size of the fused kernels
constexpr int kSpmmThreads = 256;        // workgroup size of the row-list SpMM kernel
constexpr int kWantedTileRows = 256;     // a default column slice is narrowed until tiles this large fit
constexpr int kGatherEntries = 8;        // entries per row that the gather kernel has in flight
constexpr int kGatherQuad = kSpmmThreads / 64;   // blocks that its workgroups take at a time
constexpr int kGatherSliceBytes = 128;   // a cache line: column slices of the gather kernel chosen by default, bytes
constexpr int64_t kStaticScratchBytes = (int64_t)64 << 20;   // workspace of tf_gemm_spmm_static

// Per D1 row of a tile, beside its row id: one info word.  kInfoSpill: the row is also stored to
// the D1 workspace, at the slot in the low bits (a row that the second wavefront reads).
// kInfoDirect: the row of D with the same id is fused and has exactly one stored entry, on the
// diagonal, so it is the D1 row times that entry (tile_scale) and leaves from the registers that
// hold the D1 row; kInfoZero: the row of D with the same id is empty and is stored as zeros.
// 0 for padding rows.
constexpr uint32_t kInfoSpill = 0x80000000u;
constexpr uint32_t kInfoDirect = 0x40000000u;
constexpr uint32_t kInfoZero = 0x20000000u;
// kInfoSkip (streaming first wavefront of a CSR-B plan with TF_FLAG_SKIP_UNREAD only): no row of A
// reads this D1 row, it is not computed.
constexpr uint32_t kInfoSkip = 0x10000000u;
constexpr uint32_t kInfoSlotMask = 0x0fffffffu;
// A finished D1 row in k_csr_spmm: its info word, which without row_info says that the row is stored to the workspace,
// and the slot there, which then is the row's own number (it may take more bits than an info word has).
constexpr uint32_t d1_info(bool has_info, uint32_t info) { return has_info ? info : kInfoSpill; }
constexpr int64_t d1_slot(bool has_info, uint32_t info, int64_t row) {
    return has_info ? (int64_t)(info & kInfoSlotMask) : row;
}
// Rows of S in k_csr_spmm, `nr` consecutive ones a block; every XCD takes eighths of the blocks.  Unsigned: row, block and
// entry numbers run past the last one, which may be 2^31 - 2.
struct CsrBlocks {
    uint32_t n_rows, nr;
    constexpr uint32_t count() const { return (n_rows + nr - 1) / nr; }
    constexpr uint32_t eighth() const { return (count() + kXcds - 1) / kXcds; }
    constexpr uint32_t end(uint32_t eighths) const { return eighths * eighth() < count() ? eighths * eighth() : count(); }
    constexpr bool has(uint32_t block, uint32_t v) const { return block * nr + v < n_rows; }
    constexpr uint32_t row(uint32_t block, uint32_t v) const { return has(block, v) ? block * nr + v : n_rows - 1; }
};
// The blocks that one of `waves` waves takes, which move through a range side by side: block `at`, numbered within its
// round by `place`.  Every round begins three waves further: rows with many entries sit at multiples of powers of two in
// the graphs that are made by recursion, and at a fixed place the same wave would take them all (a b c d = .57 .19 .19 .05,
// 2^20 rows, 512 waves: that wave has 25224 passes, now 5050, of which the longest row alone takes 4967).
constexpr uint32_t kCsrTurn = 3;
struct CsrWalk {
    uint32_t at, place;
    constexpr CsrWalk next(uint32_t waves) const {
        const uint32_t to = place + kCsrTurn;
        return to < waves ? CsrWalk{at + waves + kCsrTurn, to} : CsrWalk{at + kCsrTurn, to - waves};
    }
};
// Is there an entry number s (which may lie as far behind the row as another row of its block is long) in the row of
// the entries begin to end - 1?
constexpr bool has_entry(int32_t begin, int32_t end, uint32_t s) { return s < (uint32_t)(end - begin); }

// Where the D1 rows that cross tiles live in device memory: `n_sl` column slices of `sw` columns
// each (the last may be narrower in use, never in storage), slice after slice, each slice a dense
// array of `rows` rows of sw elements.  Element (slot, col) is at
// (col / sw) * rows * sw + slot * sw + col % sw.  One slice = plain row-major.  Slices are what one
// XCD of the gather kernel works on: its L2 then holds sw-wide pieces of the rows instead of whole
// rows, and the hot rows of an irregular matrix are not replicated in all eight L2 caches.
struct D1Layout {
    int32_t sw = 0, n_sl = 1;
    int64_t rows = 0;
    int64_t slice_stride() const { return rows * sw; }
    int64_t elements() const { return (int64_t)n_sl * rows * sw; }
    int64_t columns() const { return (int64_t)n_sl * sw; }
};

// Do slices of one cache line pay, `laid_out` bytes of them for rows of row_bytes?  They move that much more and read the
// entries of A once per slice; they save what an L2 then holds: `reuse` is the share of entries whose column is among as
// many others as it holds lines (Schedule::reuse).  Second wavefront, rows of 36 to 128 columns, both types, 130 points
// (slices / whole rows, us: R-MAT graph of 2^20, .44, fp32 128 columns 701 / 973, 400000, .56, 236 / 344; uniform columns, 8
// a row, 60000 rows, .44, 28.5 / 39.2; 250000, .14, 162 / 165, fp64 90 columns 283 / 265; 700000, .05, fp32 128 columns 488 /
// 458, 36 columns 275 / 214, fp64 90 columns 1013 / 727).  Below .3 the line is a fit: 0.8 % above the better way on average and 7
// at most, where slices in any case are 6 and 39; from .3 on slices gain up to 39 %, and lose only where rows are little
// longer than a line (fp32, 36 columns, 78 % more to move, up to 23 %).
inline bool line_slices_pay(int64_t laid_out, int64_t row_bytes, double reuse) {
    return reuse >= 0.3 || (double)laid_out <= (0.9 + 1.25 * reuse) * (double)row_bytes;
}

// Column slices in which the rows of a dense B are gathered: one cache line each, where rows are whole lines
// (rows of slices that begin anywhere in a line would touch more of them); `rows` rows of bcol columns,
// element (i, c) at i bcol + c whatever the slices.
inline D1Layout gather_first_slices(int dtype, int64_t rows, int64_t bcol, double reuse) {
    const int64_t es = dtype == TF_F64 ? 8 : 4;
    D1Layout l;
    l.rows = rows;
    l.sw = (int32_t)bcol;
    if (bcol * es % kGatherSliceBytes || !line_slices_pay(bcol * es, bcol * es, reuse)) return l;
    int64_t k = bcol * es / kGatherSliceBytes;
    while (k > kXcds && k % 2 == 0) k /= 2;
    if (k > kXcds) return l;
    l.n_sl = (int32_t)k;
    l.sw = (int32_t)(bcol / k);
    return l;
}

// Column slices in which a CSR B gathers rows of C: one cache line each, where rows are whole lines and a slice of C is
// not far from what an L2 holds.  The pattern of B is not known; rows of A that reach far stand for it.  (Random rows of
// eight entries, first operation, us, whole rows / slices: 20000 rows fp64 64 columns 12.0 / 8.7, 40000 fp32 128, six
// entries, 19.9 / 14.8, 60000 fp64 128 75 / 65, 100003 fp64 64 60.8 / 57.7, 100000 fp32 64 31.0 / 29.3; beyond: 200000
// rows fp32 64, five entries, 42.8 / 44.2, 300000 fp32 128 177 / 198.)
inline void csr_slices(bool far_rows, int dtype, int64_t c_rows, int64_t ccol, int32_t &n_sl, int32_t &sw) {
    const int64_t row = ccol * (dtype == TF_F64 ? 8 : 4);
    n_sl = 1;
    sw = (int32_t)ccol;
    if (!far_rows || row % kGatherSliceBytes) return;
    const int64_t k = row / kGatherSliceBytes;
    if (k < 2 || k > kXcds || c_rows * kGatherSliceBytes > ((int64_t)16 << 20)) return;
    n_sl = (int32_t)k;
    sw = (int32_t)(ccol / k);
}

// Lanes that share one row in the gather kernels: each lane owns vv columns (vv = elements per
// 16 bytes when rows are 16-byte aligned, else 1); the group is the smallest power of two of
// lanes that covers `cols` columns, at most one wave.
inline int lane_group(int cols, int vv) {
    int g = 1;
    while (g * vv < cols && g < 64) g *= 2;
    return g;
}

// Rows of `each` entries (1 to 4) that a virtual row of G lanes holds; 1: such blocks are not made.
constexpr int gather_short_rows(int each, int G) {
    const int r = each == 1 ? 8 : each == 2 ? 4 : 2;
    return each < 1 || each > 4 || G < r ? 1 : r;
}
// Waves per SIMD that the gather kernel is held to: one more spills some 40 bytes a lane (R-MAT graphs, rows of 32 and
// 64 fp32 columns, 30000 to 300000 rows: 3 to 20 % slower).
constexpr int gather_waves(int dtype) { return dtype == TF_F64 ? 4 : 5; }
// The same for rows of a caller's matrix, G lanes each: the extents and entries of 64 or 32 rows a wave take registers.
constexpr int csr_waves(int dtype, int G) { return dtype == TF_F64 ? (G == 1 ? 2 : G == 2 ? 3 : 4) : G == 1 ? 3 : 4; }

inline int elem_size(int dtype) { return dtype == TF_F64 ? 8 : 4; }
inline int vec_elems(int dtype) { return dtype == TF_F64 ? 2 : 4; }   // elements per 16 bytes

// Columns per lane where rows are gathered, for column slices of cs of the ccol columns: sixteen bytes,
// also where they are not aligned (device memory takes a 16-byte access at any element), as long as
// every slice holds one such piece.  The last piece of a slice that is no whole number of them is
// moved back so that it ends with the slice: what it shares with the piece before is computed and
// stored twice, the same bits both times.  One column per lane, as the
// kernels run for narrower slices, fetches and stores the same bytes with four times the instructions
// (fp32): A (A C) on a 45^3 stencil, 30 columns, 35.6 us against 24.5 us.
inline int lane_elems(int dtype, int64_t ccol, int64_t cs) {
    const int v = vec_elems(dtype);
    const int64_t last = ccol > 0 ? (ccol - 1) % cs + 1 : 0;
    return cs >= v && last >= v ? v : 1;
}

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// LDS layout of a fused workgroup, shared by the inspector (tile fitting) and the kernels.
//   dense B : [C slice in MFMA operand order: bcol_pad x cs16] [D1 tile: rows_pad16 x ldl]
//   sparse B: [D1 tile: rows x ldl]
// ldl is the leading dimension of the D1 tile in elements; dense-B tiles are as wide as the
// MFMA blocks that produce them and carry 16 bytes of padding per row so that the 16 rows written
// by one MFMA block start in different banks.
// Number of 16-column accumulator blocks the MFMA phase runs for a slice of cs columns
// (instantiated for 1, 2, 4 and 8 blocks) and the padded slice width that goes with it.
inline int mfma_blocks(int cs) {
    int nb = 1;
    while (nb * 16 < cs) nb *= 2;
    return nb;
}
inline int mfma_cols(int cs) { return 16 * mfma_blocks(cs); }
inline int64_t lds_ldl(int dtype, int b_is_sparse, int cs) {
    const int v = vec_elems(dtype);
    return b_is_sparse ? round_up(cs, v) : mfma_cols(cs) + v;
}
inline int64_t lds_fixed_bytes(int dtype, int b_is_sparse, int bcol, int cs) {
    if (b_is_sparse) return 0;
    const int kc = 4 * vec_elems(dtype);
    return round_up(bcol, kc) * mfma_cols(cs) * elem_size(dtype);
}
inline int lds_row_granule(int b_is_sparse) { return b_is_sparse ? 1 : kRowGranuleDense; }
// A CSR B: the workgroup first copies the extents of the tile's rows of B and up to
// kSparseEntryCap entries of each into LDS (two loads per row for the whole tile instead of a
// chain of dependent loads per row); bytes of LDS per tile row that this takes.
constexpr int kSparseEntryCap = 8;
inline int64_t lds_sparse_b_bytes_per_row(int dtype) {
    return 2 * 8 + kSparseEntryCap * (4 + (int64_t)elem_size(dtype));    // extents of two tiles
}

// The fp32 product on the bf16 matrix cores (k_gemm_split): products of some size, rows of B of up to kSplitMaxDepth columns.
// Below, the fp32 instructions of k_gemm: their C is laid out sooner and their blocks are half as many rows (whole executions on
// R-MAT graphs, us, k_gemm / k_gemm_split: 20000 rows 64 -> 64 19.2 / 19.2, 128 -> 41 21.2 / 23.6, 128 -> 128 33.8 / 35.0; 60000
// rows 8 -> 8 16.5 / 17.6, 64 -> 20 24.1 / 24.4, 16 -> 128 25.2 / 24.1, 32 -> 32 20.8 / 19.3, 128 -> 128 61.4 / 55.8).  Blocks of
// sixteen columns that a slice of cs columns takes, and the LDS for C in three parts.
constexpr int kSplitMinDepth = 16, kSplitMaxDepth = 128, kSplitMinCols = 32, kSplitMinRows = 32768;
inline bool gemm_splits(int dtype, int64_t n, int bcol, int cs) {
    return dtype == TF_F32 && n >= kSplitMinRows && bcol >= kSplitMinDepth && bcol <= kSplitMaxDepth && cs >= kSplitMinCols;
}
inline int split_col_blocks(int cs) {
    const int nb = (cs + 15) / 16;
    return nb == 5 ? 6 : nb == 7 ? 8 : nb;
}
constexpr int64_t split_lds_bytes(int steps, int nb) { return (int64_t)steps * nb * 3 * 1024 + nb * 16 * 4; }

// Whether a wave of the dense-B kernels keeps its operands of the C slice in registers: only for
// the specialised shallow depths (ks = bCol / (4 * elements per 16 bytes) steps, nb accumulator
// blocks) and at most 64 registers' worth (32 for fp64, whose B buffers are twice as large).
// The C slice then needs no LDS.
constexpr bool c_in_registers(int dtype, int nb, int ks) {
    return (ks == 2 || ks == 4) &&
           ks * (dtype == TF_F64 ? 2 : 4) * nb * (dtype == TF_F64 ? 2 : 1) <= (dtype == TF_F64 ? 32 : 64);
}
// ks as the kernels specialise it: 0 = generic loop over k.
inline int mfma_ksteps_special(int dtype, int bcol, int ccol, int cs) {
    const int v = dtype == TF_F64 ? 2 : 4;
    if (bcol % v || ccol % v || cs % v || bcol % (4 * v)) return 0;
    const int ks = bcol / (4 * v);
    return (ks == 2 || ks == 4 || ks == 8 || ks == 16) ? ks : 0;
}

// What a fused workgroup needs to know about one tile: the ids of its D1 rows, one info word per
// row (kInfo*: spill slot, direct, zero) and the diagonal entry of direct rows, in three arrays with
// the same stride for every tile, so that their addresses follow from the tile's number alone
// (the first loads of a workgroup do not wait for a descriptor); padding up to the stride repeats
// the last row, with an empty info word.  And, so that nothing in the tile waits for a
// chain of dependent loads (row list -> unit -> entries), this fixed-size descriptor plus one
// contiguous, 16-byte aligned second-phase block of s_bytes bytes (each array padded to 16 bytes):
//   TileUnit units[n_units]
//   int32    rows2[n_second]               row ids of the fused rows of D, unit after unit
//   uint16   idx[n_entries]                where the D1 row of every packed entry sits in the LDS tile,
//                                          in units of 16 bytes: the even slots of all rows first
//                                          (n_entries / 2 of them), then the odd slots
//   T        val[n_entries]
struct TileDesc {
    int64_t meta_off;      // byte offset of the block
    int32_t n_rows;        // D1 rows the tile produces
    int32_t n_units;
    int32_t n_second;      // fused rows of D that read the LDS tile (direct rows are not among them)
    int32_t n_entries;     // padded entries over all units
    int32_t s_bytes;       // size of the second-phase block
    int32_t reserved;
};
struct TileUnit {          // n_rows rows of `stride` entry slots each, from entry_base on
    int32_t entry_base;    // even
    int32_t row_begin;     // position of the unit's first row in rows2
    int32_t n_rows;
    int32_t slots;         // stride (even, low 16 bits) | real length of the longest row (high 16 bits)
};

// Dynamic LDS of a fused workgroup: two buffers of row ids (this tile's and the next one's),
// the staged second-phase block (s_lds bytes, 0 when it is read in place), the staged rows of a
// CSR B, the C slice of a dense B unless the waves hold it in registers, the D1 tile.
struct FusedLdsLayout {
    int64_t first0, first1, second, bext, bidx, bval, cslice, tile, total;
};
inline FusedLdsLayout fused_lds_layout(int dtype, int b_is_sparse, int bcol, int ccol, int cs,
                                       int max_tile_rows, int s_lds, bool need_tile = true) {
    FusedLdsLayout l{};
    const int es = elem_size(dtype);
    const int64_t rows16 = round_up(max_tile_rows, 16);       // the row id buffers are padded
    const int64_t rows_cap = round_up(max_tile_rows, lds_row_granule(b_is_sparse));
    l.first0 = 0;
    l.first1 = rows16 * 4;
    l.second = 2 * rows16 * 4;
    // staged rows of a CSR B: (first entry, length) per row for this tile and for the next one,
    // then the column indices, then the values
    l.bext = l.second + round_up(s_lds, 16);
    l.bidx = l.bext + (b_is_sparse ? 2 * round_up(rows_cap * 8, 16) : 0);
    l.bval = l.bidx + (b_is_sparse ? round_up(rows_cap * kSparseEntryCap * 4, 16) : 0);
    l.cslice = l.bval + (b_is_sparse ? round_up(rows_cap * kSparseEntryCap * es, 16) : 0);
    const int64_t cbytes = lds_fixed_bytes(dtype, b_is_sparse, bcol, cs);
    const bool c_regs = !b_is_sparse && c_in_registers(dtype, mfma_blocks(cs),
                                                       mfma_ksteps_special(dtype, bcol, ccol, cs));
    l.tile = l.cslice + (c_regs ? 0 : cbytes);
    // (a plan none of whose fused rows reads the tile keeps no tile at all)
    l.total = l.tile + (need_tile ? rows_cap * lds_ldl(dtype, b_is_sparse, cs) * es : 0);
    return l;
}
inline int64_t fused_lds_bytes(int dtype, int b_is_sparse, int bcol, int ccol, int cs,
                               int max_tile_rows, int s_lds, bool need_tile = true) {
    return fused_lds_layout(dtype, b_is_sparse, bcol, ccol, cs, max_tile_rows, s_lds, need_tile).total;
}

// One block of a packed row list: what a wave of the gather kernel works on at a time.  It holds `nr` virtual
// rows (nr = 64 lanes over the lanes of a row): rows, or the 2^k equal parts that each row of the block is cut
// into, in adjacent lane groups; or nr parts of one row that takes the four blocks of a workgroup, or several
// times that (pieces).  The list is a whole number of fours, filled up with blocks of no rows.
struct GatherBlock {
    uint32_t slot_base;    // first slot of the block: entry (slot s, virtual row v) is at (slot_base + s) nr + v
    int32_t row_begin;     // position of the block's first row in the list
    uint32_t size;         // slots of every virtual row (0: the block's rows are empty) | slots that hold an entry
                           // in all of them << 16
    uint32_t info;         // k (3 bits) | e (3 bits) | rows of the block << 6; e > 0: rows of e entries each, several to
                           // a virtual row (gather_short_rows), one after the other in its slots
    int slots() const { return (int)(size & 0xffff); }
};
// The blocks of rows that are cut over several come first; for each of them:
struct CutBlock {
    int32_t skip;          // entries of the row before the block's
    int32_t piece;         // number of the piece, over all cut rows
    int32_t row;           // number of the cut row
    int32_t first_piece;   // its first piece
    int32_t pieces;
};

// A vector whose resize() leaves the new elements uninitialised: the packed arrays are sized once
// and then written in full by the host threads, which are also the first to touch their pages.
template <typename T> struct NoInitAlloc : std::allocator<T> {
    template <typename U> struct rebind {
        using other = NoInitAlloc<U>;
    };
    template <typename U> void construct(U *p) noexcept { ::new (static_cast<void *>(p)) U; }
    template <typename U, typename... A> void construct(U *p, A &&...a) {
        ::new (static_cast<void *>(p)) U(std::forward<A>(a)...);
    }
};
template <typename T> using RawVec = std::vector<T, NoInitAlloc<T>>;

// A list of rows of A re-packed for the gather kernel.  Padding repeats the row's last column index with
// value 0; the kernel leaves it out of the sums.
struct RowPack {
    std::vector<GatherBlock> blocks;
    std::vector<int32_t> rows;           // row ids, list order
    std::vector<int32_t> lens;           // their entries
    RawVec<int32_t> idx32;               // column indices
    RawVec<unsigned char> vals;          // packed values, element size of the plan's dtype
    bool sorted = false;                 // rows were re-ordered by length
    int32_t n_pieces = 0;
    int32_t n_cut_rows = 0;              // rows cut over several blocks
    std::vector<CutBlock> cuts;          // their blocks
    int64_t n_counts = 0;                // counts of their finished pieces, per slice and column block
};

// ---- the chain in one pass, D = (A B) C (dense B) -----------------------------------------------
// A is re-packed into blocks of sixteen virtual rows: a row, or one of the 2^k equal parts that the
// rows of the block are cut into.  All virtual rows of a block have `slots` entries (padding: column
// kChainPad, value 0), stored slot after slot, sixteen entries each.
struct ChainBlock {
    uint32_t slot_base;    // first slot of the block: its entries start at 16 slot_base
    int32_t slots;         // 0: the block's rows are empty
    int32_t row_begin;     // position of the block's first row in the row list
    int32_t info;          // log2 of the parts per row (3 bits) | slots per gather pass << 3 (4 bits) |
                           // rows of the block << 7
};
struct ChainPack {
    std::vector<ChainBlock> blocks;
    std::vector<int32_t> rows;           // row ids in block order
    RawVec<int32_t> idx;
    RawVec<unsigned char> vals;
    bool early = false;                  // chain_early
};
constexpr int kChainThreads = 512;       // largest workgroup of the kernel
constexpr int kChainMaxEntries = 8;      // most entries per row in flight
constexpr int kChainSpreadDepth = 6;     // depth from which the blocks of a last round may be dealt over the workgroups
constexpr int kChainLongRow = 1024;      // longest row a block takes
constexpr int kChainMaxCut = 4;          // log2 of the most parts that a row is cut into
constexpr int32_t kChainPad = -1;        // the column of a padding entry: zeros are read in the place of a row of B
constexpr int kChainSpareSlots = 2 * kChainMaxEntries;   // zero slots behind the last block (entries are fetched ahead)
constexpr int kChainZeroRows = 16;       // copies of a row of zeros, which padding reads, behind the values
constexpr int kChainRowBytes = 1024;     // longest row of B
// 16-byte pieces of a row of B per lane: ceil(bCol / (4 V)) rounded up to a depth the kernel is
// instantiated for; 0 = none.  The depths end at 128 columns: there the kernel takes 238 of the 256 registers
// of a wave in fp64, with two entries in flight per row, and 234 in fp32, with three; deeper instances were not
// built.  Wider rows of B take the two wavefronts (2D stencil 512^2, -> 64, us at 128, 132 and 129 columns: fp32
// 61, 94, 133; fp64 at 128, 130 and 129: 133, 261, 288).
constexpr int kChainDepths32[] = {1, 2, 3, 4, 6, 8}, kChainDepths64[] = {2, 4, 6, 8, 12, 16};
inline int chain_ksteps(int dtype, int64_t bcol) {
    const int v = vec_elems(dtype);
    if (bcol < v) return 0;
    for (int k = 0; k < 6; ++k) {
        const int ks = dtype == TF_F64 ? kChainDepths64[k] : kChainDepths32[k];
        if (bcol <= (int64_t)4 * v * ks) return ks;
    }
    return 0;
}
static_assert(4 * 16 * kChainDepths32[5] <= kChainRowBytes && 4 * 16 * kChainDepths64[5] <= kChainRowBytes,
              "a copy of the zeros is as long as the longest row of B");
// The depth below `ks`: pieces up to there are whole in every row that takes depth ks.
constexpr int chain_ksteps_below(int dtype, int ks) {
    int below = 0;
    for (int k = 0; k < 6; ++k) {
        const int d = dtype == TF_F64 ? kChainDepths64[k] : kChainDepths32[k];
        if (d < ks) below = d;
    }
    return below;
}
// Whether a wave sends out the next block's first gathers before it multiplies (k_gather_gemm, EARLY): fp64 at depth 8, whose rows
// take two trips to memory with up to eight entries and have little to multiply meanwhile.  It pays where rows have few
// entries and B does not fit the L2s, from 24 MiB at up to five entries a row, 36 MiB at up to seven; longer rows take more passes
// of four than of five, and where B and D are more than the last-level cache holds, rows gathered twice come from memory twice.
// us, all gathers after the stores / the first ones early: 2D stencils 200^2 64 -> 20 11.3 / 11.7, 225^2 64 -> 64 21.0 / 20.0, 512^2 64 ->
// 20 47.5 / 43.9, 50 -> 23 47.1 / 42.1, 64 -> 64 64.8 / 63.4, 700^2 (329 MB) 64 -> 20 85.7 / 91.6, (500 MB) 64 -> 64 136 / 142; 3D 36^3 64 -> 20
// 14.3 / 15.0, 40^3 57 -> 32 18.8 / 19.0, 48^3 64 -> 64 38.0 / 35.7, 64^3 64 -> 64 83.3 / 72.1; bands of 60000 rows, 64 -> 20, of 5 15.6 /
// 14.8, of 7 16.4 / 17.0, of 9 18.2 / 19.0.  Before the gathers came after the stores at all, three entries a pass: 512^2 64 -> 20 45.2,
// 50 -> 23 43.4, 64 -> 64 64.1, 64^3 64 -> 64 74.9.
constexpr int64_t kChainEarlyMost = (int64_t)300 * 1000 * 1000;
inline bool chain_early(int dtype, int ks, int64_t n, int64_t nnz, int64_t bcol, int64_t ccol) {
    if (dtype != TF_F64 || ks != 8 || nnz > 7 * n) return false;
    return n * bcol * 8 >= (int64_t)(nnz <= 5 * n ? 24 : 36) << 20 && n * (bcol + ccol) * 8 <= kChainEarlyMost;
}
// Entries per row whose gathers are in flight at once (about 24 pieces of 16 bytes per lane; fp64 at depths 8 and 12, whose waves
// have 256 registers, 40 and 36, 32 early: bands, 64 -> 64 84 -> 80 us, 96 -> 96 134 -> 126).
constexpr int chain_entries(int dtype, int ks, bool early) {
    return early ? 4 : ks <= 2 ? 8 : ks == 3 ? 6 : ks == 4 ? 5 : ks == 8 && dtype == TF_F64 ? 5 : ks <= 8 || (ks == 12 && dtype == TF_F64) ? 3 : 2;
}
// Waves per SIMD that the kernel is held to: where a third one costs no spilled registers (fp64 at depth 2 with
// four blocks of columns: held to three it spills 12 bytes a lane; bands and 3D stencils, 16 -> 64, us
// with three and two: 264964 rows of 5 32.9 / 30.9, 60^3 29.9 / 27.5, 439631 rows of 12, 8 -> 64, 63.7 / 61.3).
constexpr int chain_waves(int dtype, int ks, int nbc) {
    return dtype == TF_F64 ? (ks == 2 && nbc < 4 ? 3 : 2) : ks <= 6 ? 3 : 2;
}
// Blocks of sixteen columns of D that are multiplied together: the count (3 or 4, or all of them)
// that wastes the fewest blocks; two at the largest depth, where the registers end.
inline int chain_col_blocks(int ks, int64_t ccol) {
    const int64_t nb = (ccol + 15) / 16;
    if (ks >= 16) return nb > 1 ? 2 : 1;
    if (nb <= 4) return (int)nb;
    return (nb + 2) / 3 * 3 < (nb + 3) / 4 * 4 ? 3 : 4;
}
// LDS per wave (see k_gather_gemm): loads of 64 entries per pass, k steps per change of lanes, blocks of
// sixteen columns that leave together, and what that comes to in bytes.
constexpr int chain_entry_loads(int dtype, int ks, bool early) { return (chain_entries(dtype, ks, early) + 3) / 4; }
// (whole loads are put into LDS; fp64 at depth 8, whose C may leave no room for them, keeps to the entries of a pass: the test
// for them costs 2 to 5 % where launches are small)
constexpr int chain_entry_slots(int dtype, int ks, bool early) {
    return dtype == TF_F64 && ks == 8 ? 16 * chain_entries(dtype, ks, early) : 64 * chain_entry_loads(dtype, ks, early);
}
constexpr int chain_exchange(int ks) { return ks < 4 ? ks : ks < 16 ? 4 : 2; }
constexpr int chain_store_blocks(int dtype, int ks, int nbc) {
    return dtype == TF_F32 ? nbc : ks < 16 && nbc % 2 == 0 ? 2 : 1;
}
constexpr int chain_exchange_bytes(int dtype, int ks, int nbc) {
    const int in = chain_exchange(ks) * 1024;
    const int out = 16 * (chain_store_blocks(dtype, ks, nbc) * 16 * (dtype == TF_F64 ? 8 : 4) + 16);
    return in > out ? in : out;
}
constexpr int64_t chain_wave_lds(int dtype, int ks, int nbc, bool early) {
    return chain_exchange_bytes(dtype, ks, nbc) + 64 + chain_entry_slots(dtype, ks, early) * (8 + (dtype == TF_F64 ? 8 : 4));
}
// Whether the kernel multiplies on the bf16 matrix cores, by operands split in three: rows of B of more than 48 columns and rows
// of D of more than sixteen (shorter rows of B: three parts of C take longer to lay out than is saved; one block of columns:
// splitting the rows does; us, fp32 instructions / split, 2D stencil 120^2: 8 -> 8 5.1 / 6.1, 16 -> 64 5.7 / 7.0, 32 -> 32 5.5 /
// 6.6, 50 -> 23 6.4 / 6.1, 128 -> 32 8.8 / 7.8; 200^2: 56 -> 16 6.4 / 7.6, 128 -> 16 9.0 / 9.9, 128 -> 20 12.0 / 10.8; 353^2: 64 -> 16 11.6 /
// 13.0, 64 -> 20 16.0 / 15.0).
constexpr bool chain_splits(int dtype, int ks, int nbc) { return dtype == TF_F32 && ks >= 4 && nbc > 1; }
// LDS of a group of blocks of columns of C: fp64 as the multiplications take it, fp32 in three parts of bf16 with the largest
// number of each column.
constexpr int64_t chain_group_lds(int dtype, int ks, int nbc) {
    return chain_splits(dtype, ks, nbc) ? (int64_t)nbc * ((ks + 1) / 2 * 3 * 1024 + 64) : (int64_t)nbc * ks * 1024;
}
// What decides whether a plan may take the one pass: C, and for each wave of the largest workgroup the exchange and 64 or 128
// entries.  The kernel takes as much or, for entries of fp64 at depth 8, 256 bytes more a wave, for which there is room
// (blocks of columns are 8 KiB there); C in three parts may take more, it is then multiplied by in several workgroups.
inline int64_t chain_lds_bytes(int dtype, int64_t bcol, int64_t ccol) {
    const int ks = chain_ksteps(dtype, bcol);
    const int64_t nb = (ccol + 15) / 16, nbc = chain_col_blocks(ks, ccol);
    return (nb + nbc - 1) / nbc * nbc * 16 * ks * 4 * vec_elems(dtype) * elem_size(dtype) +
           kChainThreads / 64 * (chain_exchange_bytes(dtype, ks, (int)nbc) + 64 + (ks <= 4 ? 128 : 64) * (8 + elem_size(dtype)));
}

// Host-side schedule produced by the inspector.
struct Schedule {
    int64_t n = 0, nnz = 0;
    int32_t t = 0;                 // step-1 uniform tile size
    int32_t col_slice = 0, n_slices = 1;
    int64_t n_coarse_tiles = 0;
    std::vector<int32_t> tile_first_ptr, first_rows;      // first_rows: plain row ids
    std::vector<int32_t> tile_second_ptr, second_rows;
    std::vector<int32_t> wf1_unit_ptr, wf1_rows;
    std::vector<uint8_t> spill;
    std::vector<TileDesc> tile_desc;                      // one per tile, see TileDesc
    // the tiles' second-phase blocks, back to back (not zero-filled on allocation: the host threads
    // that copy the blocks in are the first to touch its pages)
    std::unique_ptr<unsigned char[]> tile_meta;
    size_t tile_meta_bytes = 0;
    std::vector<int32_t> tile_first;                      // the tiles' row ids, first_stride ints per tile
    std::vector<uint32_t> tile_info;                      // info word per D1 row of a tile (kInfo*), same stride
    RawVec<unsigned char> tile_scale;                     // diagonal entry of the direct rows (plan's dtype), same stride; empty when there are none
    std::vector<int32_t> spill_slot;                      // per row: its slot in the D1 workspace, -1 when not spilled
    D1Layout d1;                                          // workspace of the fused path (rows = spilled rows)
    int64_t n_direct_rows = 0;                            // fused rows that leave from registers (diagonal-only or empty)
    int64_t n_lds_rows = 0;                               // fused rows computed out of the LDS tile
    // When no fused row reads the LDS tile the first wavefront streams through the rows without
    // tiles: the info words and diagonal entries again, indexed by row (empty otherwise).
    std::vector<uint32_t> row_info;
    RawVec<unsigned char> row_scale;
    bool streaming = false;
    bool automatic = false;        // the caller left the tiling to the library
    bool far_rows = false;         // rows reach far from the diagonal (a graph), see build_schedule
    double far_b_share = 0.0;      // share of the entries whose row of B is more than 1 MiB away from the row's own
    bool grown_tiles = false;      // tiles grown along the dependence graph
    int64_t n_demoted_rows = 0;    // rows that a tile could have fused but that were left to the second wavefront
    int32_t first_stride = 0;                             // largest tile, in rows, rounded up to 16
    int64_t second_block_cap = 0;                         // largest second-phase block, bytes
    bool second_block_in_lds = true;                      // it fits beside the largest tile
    int64_t lds_meta_bytes_per_row = 0;                   // part of lds_bytes_per_row: row ids + estimate of the second-phase block
    RowPack wf1;                   // wf1_rows re-packed
    RowPack all;                   // all rows re-packed (unfused baseline)
    bool plain_pair = false;       // CSR B: the fused calls run the two operations over all rows, see plain_pair_is_faster
    ChainPack chain;               // all rows re-packed for the one-pass chain; no blocks: not used
    // The chain as Y = A B, D = Y C (see choose_gather_first).
    bool gather_first = false;
    double reuse = 1.0;                    // (rows that reach far) share of entries of A whose column is among those of
                                           // as many other entries as an L2 holds cache lines
    bool gather_first_shares = false;      // Y is gathered with `all`, else with `gf`
    RowPack gf;
    std::vector<uint32_t> gf_info;         // info word per row of Y: its row of D, or zeros
    int64_t n_fused_rows = 0, n_spill_rows = 0, fused_nnz = 0;
    int64_t max_tile_rows = 0;
    int64_t lds_fixed_bytes = 0, lds_bytes_per_row = 0, fast_mem_bytes = 0;
    int32_t lds_row_granule = 1;
    double eq2_cost_max = 0.0;
};

struct InspectorInput {
    int64_t n, nnz;
    const int32_t *rowptr, *colidx;   // host
    const void *vals;                 // host, element size of dtype
    int64_t bcol, ccol;
    int32_t b_is_sparse;
    int32_t dtype;
    int32_t ct_size, p;
    int64_t fast_mem_bytes;
    int32_t col_slice;
    uint32_t flags;
    int32_t gather_slices;            // column slices of the D1 workspace and of the gather kernel; 0 = chosen here
    int32_t n_cu;                     // compute units of the device the plan will run on
    bool whole_fast_mem;              // fast_mem_bytes is the device's own, not the caller's
};

// Builds the schedule; returns TF_OK or an error with a message in `err`.
tf_status build_schedule(const InspectorInput &in, Schedule &out, std::string &err);
// The packed copy of all rows of A that the unfused baseline's second operation runs on
// (Schedule::all).  Not part of the fused schedule and not counted in its time.
void build_baseline_pack(const InspectorInput &in, Schedule &s);
// Decides whether the fused calls of the plan run the chain in one pass, and packs A for it (entries =
// false: the blocks only).
void build_chain_pack(const InspectorInput &in, Schedule &s, bool entries);
// Whether the fused calls of a CSR-B plan run the plain pair of operations.
bool plain_pair_is_faster(const InspectorInput &in, const Schedule &s);
// Decides whether they run it as Y = A B, D = Y C (Schedule::gather_first).
void choose_gather_first(const InspectorInput &in, Schedule &s);
// Packs A for that (have_all: `all` is packed).
void build_gather_first(const InspectorInput &in, Schedule &s, bool have_all);


// ---------------------------------------------------------------- device launch interface

struct CsrDev {
    const int32_t *rowptr = nullptr;
    const int32_t *colidx = nullptr;
    const void *vals = nullptr;
};

struct PackDev {
    const GatherBlock *blocks = nullptr;
    const int32_t *rows = nullptr, *lens = nullptr, *idx = nullptr;
    const void *vals = nullptr;
    const CutBlock *cuts = nullptr;
};

struct FusedLaunch {
    int32_t dtype;
    int32_t n_tiles, n_slices, cs, ccol, bcol;
    int32_t rows_cap;                 // largest tile, in rows, rounded up to 16
    int32_t tile_rows;                // largest tile, in rows, rounded up to the tile's row granule
    int32_t s_cap;                    // largest second-phase block, bytes (multiple of 16)
    int32_t s_in_lds;                 // 1: second-phase blocks are staged in LDS, 0: read in place
    int64_t lds_bytes;                // dynamic LDS of the launch
    const TileDesc *tile_desc;
    const unsigned char *tile_meta;
    const int32_t *tile_first;        // row ids of tile v at tile_first + v * first_stride
    const uint32_t *tile_info;        // info words (kInfo*), same indexing
    const void *tile_scale;           // diagonal entries of direct rows, same indexing; nullptr: no direct rows
    int32_t first_stride;
    int32_t need_tile;                // 0: no tile of the plan has fused rows that read the LDS tile
    int32_t n_cu;                     // compute units of the device
    const void *B;                    // dense B (gemm) or nullptr
    CsrDev Bs;                        // sparse B (spmm)
    const void *C;
    int32_t c_ldk, c_ldc;             // dense B: element (k, c) of the multiplier is C[k c_ldk + c c_ldc]
    void *D;
    void *D1;
    int32_t d1_sw_shift, d1_sw_mask;  // column -> (slice, offset) of the D1 workspace (one slice: 31, 0x7fffffff)
    int32_t d1_sw;
    int64_t d1_slice_stride;          // elements
};

// Y[row] = sum over the packed entries of the row of val * X[idx].
struct PackedSpmmLaunch {
    int64_t x_slice_stride;           // elements between the slices of X
    int32_t n_xs, sw;                 // column slices (1 to 8; each XCD handles n_xs eighths of one or two) of sw columns
    int32_t ldx;                      // elements between the rows of a slice
    int32_t n_blocks, n_cut_blocks;
    int32_t ccol;
    int32_t contiguous;               // 1: neighbouring blocks share an XCD; 0: round robin
    int32_t read_next;                // 1: the next launch reads Y
    int32_t few_waves;                // 1: most rows of X come from beyond the L2
    int32_t dtype;
    void *partial;                    // sums of the pieces of cut rows: [piece][slice][sw]
    uint32_t *arrived;                // pieces of a cut row that are done: [cut row][slice][column block], zeros between launches
    PackDev pack;                     // indices: rows (slots) of X
    const void *X;                    // D1 workspace in the layout above, or a dense B
    void *Y;                          // row-major, ccol columns
    int32_t wide;                     // 1: X spans 4 GiB or more (64-bit operand offsets)
    int32_t n_cu;                     // compute units of the device
};

// Y[j] = S[j, :] X for a caller-supplied CSR matrix S.
struct CsrSpmmLaunch {
    int64_t y_slice_stride;
    int32_t n_rows;
    int32_t n_xs, x_sw;               // column slices (1 to 8) of x_sw columns in which rows of X are gathered
    int32_t ccol;
    int32_t y_sw_shift, y_sw_mask, y_sw;   // D1 workspace layout: slices of y_sw columns
    int32_t dtype;
    CsrDev S;
    const void *X;                    // row-major, ccol columns
    void *Y;
    const uint32_t *row_info;         // as in GemmLaunch
    const void *row_scale;
    void *D;
    int64_t x_bytes;
    int32_t mean_len;                 // entries per row of S
    int32_t n_cu;                     // compute units of the device
};

struct GemmLaunch {
    int32_t dtype;
    int64_t n;
    int32_t bcol, ccol, cs, n_slices;
    int32_t n_cu;                     // compute units of the device
    const void *B, *C;
    int32_t c_ldk, c_ldc;             // element (k, c) of the multiplier is C[k c_ldk + c c_ldc]
    void *D1;                         // workspace layout: slices of d1_sw columns
    int32_t d1_sw_shift, d1_sw_mask, d1_sw;
    int32_t d1_cols;                  // columns of the workspace, cCol or more: the products' zeros fill what is padding
    int64_t d1_slice_stride;
    // first wavefront of a plan without an LDS tile (else nullptr): info word per row (kInfo*),
    // diagonal entry of the direct rows (nullptr: none), and D
    const uint32_t *row_info;
    const void *row_scale;
    void *D;
};

// (n, which the kernel needs last, stands first: its other numbers are then fetched by one round of scalar loads;
// in an order where that took two, a band of 4096 rows, fp64 32 -> 32, took 6.09 us in the place of 5.94)
struct ChainLaunch {
    int64_t n;
    int32_t n_blocks, n_groups, groups_per_wg;   // (the column groups are set by the launcher)
    int32_t bcol, ccol;
    int32_t c_transposed;             // C is cCol x bCol
    int32_t dtype;
    int32_t n_cu;
    const ChainBlock *blocks;
    const int32_t *rows;
    const int32_t *idx;
    const void *vals;
    const void *zeros;                // kChainZeroRows x kChainRowBytes
    const void *B, *C;
    void *D;
    int64_t lds_limit;                // of a workgroup
    int32_t early;                    // chain_early
    int32_t whole_rounds;             // (set by the launcher) rounds of blocks in their order; the rest is dealt out
};

// Each returns hipError_t as int (0 = success).  `stream` is a hipStream_t.
int launch_fused_gemm_spmm(const FusedLaunch &a, void *stream);
int launch_fused_spmm_spmm(const FusedLaunch &a, void *stream);
int launch_packed_spmm(const PackedSpmmLaunch &a, void *stream);
int launch_csr_spmm(const CsrSpmmLaunch &a, void *stream);
int launch_gemm(const GemmLaunch &a, void *stream);
int launch_gemm_split(const GemmLaunch &a, void *stream);     // where gemm_splits
int launch_chain(const ChainLaunch &a, void *stream);

}  // namespace tf
