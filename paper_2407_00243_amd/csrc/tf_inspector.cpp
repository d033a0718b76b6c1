// Inspector: the tile fusion scheduler (paper Section 3.1, Algorithm 1) for one GPU.
//
// Step 1 forms uniform tiles of t consecutive rows and fuses a row of the second operation
// into the tile that produces the same row range exactly when every column index of that row
// of A lies inside the range.  Step 2 halves every tile whose fast-memory footprint exceeds
// the budget.  The GPU additions are the spill set (D1 rows that a second-wavefront row
// reads and that therefore must also reach device memory) and the packed blocks of the second
// wavefront (the `balance` routine of Algorithm 1, read as: spread the leftover rows over waves, a
// block at a time; rows too long for a block are cut over a workgroup's four or several times that).
//
// Pure host code: no HIP calls.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <numeric>
#include <thread>

#include "tf_internal.h"

// Section timings on stderr, for profiling the inspector on its own (compile with -DTF_TIMING).
#ifdef TF_TIMING
#include <cstdio>
#define TF_TICK(label)                                                                          \
    do {                                                                                        \
        const auto tf_now = std::chrono::steady_clock::now();                                   \
        std::fprintf(stderr, "  [inspector] %-28s %8.2f ms\n", label,                           \
                     std::chrono::duration<double>(tf_now - tf_tick).count() * 1e3);            \
        tf_tick = tf_now;                                                                       \
    } while (0)
#else
#define TF_TICK(label)
#endif

namespace tf {

namespace {

struct Range {
    int64_t i0, i1;
};

int64_t tile_footprint(const Schedule &s, int64_t rows) {
    return s.lds_fixed_bytes + round_up(rows, s.lds_row_granule) * s.lds_bytes_per_row;
}

// Step 2 for one coarse tile: halve (left half gets floor(rows / 2)) until the footprint fits.
void split_tile(const Schedule &s, Range r, bool allow_split, std::vector<Range> &out) {
    const int64_t rows = r.i1 - r.i0;
    if (!allow_split || rows <= 1 || tile_footprint(s, rows) <= s.fast_mem_bytes) {
        out.push_back(r);
        return;
    }
    const int64_t mid = r.i0 + rows / 2;
    split_tile(s, Range{r.i0, mid}, allow_split, out);
    split_tile(s, Range{mid, r.i1}, allow_split, out);
}

}  // namespace

namespace {

struct PackRules {
    int nr;              // virtual rows of a block
    int64_t longest;     // most slots of a virtual row: rows of more than nr times that take several blocks
    int counts;          // counts of finished pieces per cut row (slices x column blocks)
};

// Host threads for per-tile or per-unit work: one for small matrices, else up to 16.
int host_threads(int64_t nnz, int64_t n_items, int64_t min_items_per_thread) {
    if (nnz < ((int64_t)1 << 18) || n_items < 4 * min_items_per_thread) return 1;
    unsigned hw = std::min(16u, std::max(1u, std::thread::hardware_concurrency()));
    if (const char *e = std::getenv("TF_HOST_THREADS")) {      // a cap set by the caller's environment
        const long k = std::strtol(e, nullptr, 10);
        if (k >= 1) hw = (unsigned)std::min<long>(k, 16);
    }
    return (int)std::min<int64_t>(hw, n_items / min_items_per_thread);
}

// Runs fn(v) for v in [0, count) on `nthreads` host threads, each with a contiguous range (fn
// writes to places of its own v only, so the outcome does not depend on the thread count).
template <typename Fn> void for_each_item(int64_t count, int nthreads, Fn fn) {
    if (nthreads <= 1) {
        for (int64_t v = 0; v < count; ++v) fn(v);
        return;
    }
    std::atomic<bool> failed{false};
    std::vector<std::thread> pool;
    for (int th = 0; th < nthreads; ++th)
        pool.emplace_back([&, th] {
            try {
                for (int64_t v = count * th / nthreads; v < count * (th + 1) / nthreads; ++v) fn(v);
            } catch (...) {
                failed = true;
            }
        });
    for (std::thread &t : pool) t.join();
    if (failed) throw std::bad_alloc();
}

// Re-packs the rows `list` of the CSR matrix into blocks of equal slots (see RowPack).  local(c) maps a column
// index to what the kernel should index its operand with.  First the blocks are cut (row lengths only), then
// their entries are filled in, block by block on the host threads: a block's place follows from the cuts.
template <typename LocalFn>
void pack_rows(const int32_t *rowptr, const int32_t *colidx, const unsigned char *vals, int es,
               std::vector<int32_t> list, const PackRules &rules, LocalFn local, RowPack &out) {
    out = RowPack();
    const int64_t count = (int64_t)list.size(), nr = rules.nr;
    std::vector<int32_t> &lens = out.lens;
    lens.resize((size_t)count);
    int64_t real = 0, longest = 0, shortest = 0, padded = 0;
    bool empty_inside = false;
    // rows that are measured against each other: those of a workgroup, up to 64 in long lists (a block of one
    // row is never padded, but an XCD that takes the long rows of an unsorted list holds the others up: R-MAT
    // graph of 300000 rows, fp64, 128 columns, one slice, 1702 us, sorted 448)
    int64_t window = std::min<int64_t>(64, nr * kGatherQuad);
    while (2 * window <= std::min<int64_t>(64, (count + 1023) / 1024)) window *= 2;
    auto measure = [&]() {
        real = longest = padded = 0;
        shortest = INT32_MAX;
        empty_inside = false;
        for (int64_t p0 = 0; p0 < count; p0 += window) {
            const int64_t p1 = std::min(count, p0 + window);
            int64_t mx = 0;
            for (int64_t q = p0; q < p1; ++q) {
                const int32_t j = list[(size_t)q], l = rowptr[j + 1] - rowptr[j];
                lens[(size_t)q] = l;
                real += l;
                mx = std::max<int64_t>(mx, l);
                shortest = std::min<int64_t>(shortest, l);
                empty_inside = empty_inside || (l > 0 && q > 0 && lens[(size_t)q - 1] == 0);
            }
            longest = std::max(longest, mx);
            padded += mx * (p1 - p0);
        }
    };
    measure();
    // empty rows last, so that no block mixes them with rows that need padding entries
    if (empty_inside) {
        std::stable_partition(list.begin(), list.end(), [&](int32_t j) { return rowptr[j + 1] > rowptr[j]; });
        measure();
    }
    // re-order by length when rows of equal length in every window would cost over 15 %: longest first, rows of one length in their given
    // order; by counting when the lengths are a small range, else by comparison
    if (padded > real + real * 15 / 100) {
        if (longest <= 4 * count + 1024) {
            std::vector<int64_t> start((size_t)longest + 2, 0);
            for (int32_t l : lens) ++start[(size_t)(longest - l) + 1];
            for (size_t b = 1; b < start.size(); ++b) start[b] += start[b - 1];
            std::vector<int32_t> by_len((size_t)count);
            for (int64_t q = 0; q < count; ++q)
                by_len[(size_t)start[(size_t)(longest - lens[(size_t)q])]++] = list[(size_t)q];
            list.swap(by_len);
        } else {
            std::stable_sort(list.begin(), list.end(), [&](int32_t a, int32_t b) {
                return rowptr[a + 1] - rowptr[a] > rowptr[b + 1] - rowptr[b];
            });
        }
        for (int64_t q = 0; q < count; ++q) lens[(size_t)q] = rowptr[list[(size_t)q] + 1] - rowptr[list[(size_t)q]];
        out.sorted = true;
    }
    out.rows = std::move(list);
    // rows cut over several blocks come first, in whole quads: pieces of equal length, and equal blocks of whole
    // slots inside them, so that only the last ones are padded
    const int64_t one_block = nr * rules.longest, quad = one_block * kGatherQuad;
    int log_nr = 0;
    while (1 << log_nr < nr) ++log_nr;
    if (longest > one_block)
        for (int64_t pos = 0; pos < count; ++pos) {
            const int64_t len0 = lens[(size_t)pos];
            if (len0 <= one_block) {
                if (out.sorted) break;
                continue;
            }
            const int64_t pieces = (len0 + quad - 1) / quad;
            const int64_t slots = (len0 + pieces * nr * kGatherQuad - 1) / (pieces * nr * kGatherQuad);
            GatherBlock b{};
            b.row_begin = (int32_t)pos;
            b.info = (uint32_t)log_nr | 1u << 6;
            CutBlock cut{0, 0, out.n_cut_rows++, out.n_pieces, (int32_t)((len0 + slots * nr * kGatherQuad - 1) / (slots * nr * kGatherQuad))};
            for (int64_t k = 0; k < len0;) {
                cut.piece = out.n_pieces++;
                for (int m = 0; m < kGatherQuad; ++m, k += slots * nr) {
                    const int64_t l = std::max<int64_t>(0, std::min(slots * nr, len0 - k)), here = (l + nr - 1) / nr;
                    b.size = (uint32_t)(here | std::max<int64_t>(0, l - (nr - 1) * here) << 16);
                    cut.skip = (int32_t)std::min(k, len0);
                    out.blocks.push_back(b);
                    out.cuts.push_back(cut);
                }
            }
        }
    // parts that the other rows are cut into inside their block (log2)
    auto cut_of = [&](int64_t l) {
        int c = 0;
        while ((l + (1 << c) - 1) >> c > rules.longest && c < log_nr) ++c;
        return c;
    };
    const size_t first_whole = out.blocks.size();
    int64_t pos = 0;
    if (!out.sorted && shortest > 0 && real > 4 * count && longest <= rules.longest) {
        // (the plain case, on the host threads: as many rows in every block)
        out.blocks.resize((size_t)((count + nr - 1) / nr));
        pos = count;
        for_each_item((int64_t)out.blocks.size(), host_threads(real, count, 32768), [&](int64_t k) {
            const auto at = lens.begin() + k * nr, end = lens.begin() + std::min(count, (k + 1) * nr);
            out.blocks[(size_t)k].row_begin = (int32_t)(k * nr);
            out.blocks[(size_t)k].size = (uint32_t)*std::max_element(at, end) | (uint32_t)*std::min_element(at, end) << 16;
            out.blocks[(size_t)k].info = (uint32_t)(end - at) << 6;
        });
    }
    while (pos < count) {
        const int64_t len0 = lens[(size_t)pos];
        if (len0 > one_block) {
            ++pos;
            continue;
        }
        // rows of one to four entries: as many as the slots of a pass hold, where enough of them follow each other
        const int64_t together = gather_short_rows((int)std::min<int64_t>(len0, 5), 64 / (int)nr);
        if (together > 1) {
            int64_t run = 1;
            while (run < nr * together && pos + run < count && lens[(size_t)(pos + run)] == len0) ++run;
            if (2 * run > nr * together || (run > nr && pos + run == count)) {
                GatherBlock b{};
                b.row_begin = (int32_t)pos;
                b.size = (uint32_t)(together * len0) * 0x10001u;
                b.info = (uint32_t)len0 << 3 | (uint32_t)run << 6;
                out.blocks.push_back(b);
                pos += run;
                continue;
            }
        }
        const int c = cut_of(len0);
        int64_t mx = len0, mn = len0, take = 1;
        while (take < nr >> c && pos + take < count) {
            const int64_t ln = lens[(size_t)(pos + take)];
            if ((ln == 0) != (len0 == 0) || ln > one_block || (ln != len0 && cut_of(ln) != c)) break;
            mx = std::max(mx, ln);
            mn = std::min(mn, ln);
            ++take;
        }
        const int64_t slots = (mx + (1 << c) - 1) >> c;
        GatherBlock b{};
        b.row_begin = (int32_t)pos;
        b.size = (uint32_t)(slots | std::max<int64_t>(0, mn - ((1 << c) - 1) * slots) << 16);
        b.info = (uint32_t)c | (uint32_t)take << 6;
        out.blocks.push_back(b);
        pos += take;
    }
    if (out.sorted) {
        // (rows cut into parts have half of a part's slots or more, whole rows come in their order)
        size_t end = first_whole;
        while (end < out.blocks.size() && out.blocks[end].slots() * 2 >= rules.longest) ++end;
        std::stable_sort(out.blocks.begin() + (int64_t)first_whole, out.blocks.begin() + (int64_t)end,
                         [](const GatherBlock &x, const GatherBlock &y) { return x.slots() > y.slots(); });
    }
    while (out.blocks.size() % kGatherQuad) out.blocks.push_back(GatherBlock{});
    int64_t slot = 0;
    for (GatherBlock &b : out.blocks) {
        b.slot_base = (uint32_t)slot;
        slot += b.slots();
    }
    out.n_counts = (int64_t)out.n_cut_rows * rules.counts;
    // spare entries behind the last block: the kernel fetches passes ahead, and whole passes
    const int64_t end = slot * nr, spare = std::max<int64_t>(64, 2 * kGatherEntries * nr);
    out.idx32.resize((size_t)(end + spare));
    out.vals.resize((size_t)(end + spare) * es);
    std::memset(out.idx32.data() + end, 0, (size_t)spare * 4);
    std::memset(out.vals.data() + (size_t)end * es, 0, (size_t)spare * es);
    auto fill = [&](auto tag) {
        typedef decltype(tag) T;
        const T *from = reinterpret_cast<const T *>(vals);
        T *to = reinterpret_cast<T *>(out.vals.data());
        auto fill_block = [&](const GatherBlock &b) {
            const int64_t slots = b.slots(), at = &b - out.blocks.data();
            if (slots == 0) return;
            const int c = (int)(b.info & 7), each = (int)(b.info >> 3 & 7), n_rows = (int)(b.info >> 6);
            const int64_t skip = at < (int64_t)out.cuts.size() ? out.cuts[(size_t)at].skip : 0;
            if (each) {
                int32_t *ip = out.idx32.data() + (int64_t)b.slot_base * nr;
                T *vp = to + (int64_t)b.slot_base * nr;
                const int together = (int)slots / each;
                for (int s = 0; s < (int)slots; ++s)
                    for (int v = 0; v < nr; ++v) {
                        const int ri = v * together + s / each;        // (past the block's end: not stored)
                        const int64_t k = rowptr[out.rows[(size_t)(b.row_begin + std::min(ri, n_rows - 1))]] + s % each;
                        *ip++ = (int32_t)local(colidx[k]);
                        *vp++ = from[k];
                    }
                return;
            }
            if (nr == 1 && (int64_t)(b.size >> 16) == slots) {
                const int64_t k0 = rowptr[out.rows[(size_t)b.row_begin]] + skip;
                for (int64_t s = 0; s < slots; ++s) out.idx32[(size_t)(b.slot_base + s)] = (int32_t)local(colidx[k0 + s]);
                std::memcpy(to + b.slot_base, from + k0, (size_t)slots * sizeof(T));
                return;
            }
            const int32_t *col[64];
            const T *value[64];
            int64_t n_real[64];
            for (int v = 0; v < nr; ++v) {
                // (virtual rows past the block's end repeat its last row without its values; they are not stored)
                const int32_t j = out.rows[(size_t)(b.row_begin + std::min(v >> c, n_rows - 1))];
                const int64_t k1 = rowptr[j + 1], k0 = rowptr[j] + skip + (v & ((1 << c) - 1)) * slots;
                n_real[v] = (v >> c) < n_rows ? std::max<int64_t>(0, std::min(slots, k1 - k0)) : 0;
                // (padding names the row's last column)
                col[v] = n_real[v] > 0 ? colidx + k0 : colidx + k1 - 1;
                value[v] = n_real[v] > 0 ? from + k0 : from;
            }
            int32_t *ip = out.idx32.data() + (int64_t)b.slot_base * nr;
            T *vp = to + (int64_t)b.slot_base * nr;
            int64_t s = 0;
            const int used = n_rows << c;
            for (; s < (int64_t)(b.size >> 16); ++s, ip += nr, vp += nr) {
                for (int v = 0; v < used; ++v) {
                    ip[v] = (int32_t)local(col[v][s]);
                    vp[v] = value[v][s];
                }
                for (int v = used; v < nr; ++v) {
                    ip[v] = (int32_t)local(col[v][0]);
                    vp[v] = T(0);
                }
            }
            for (; s < slots; ++s)
                for (int v = 0; v < nr; ++v) {
                    const bool in = s < n_real[v];
                    *ip++ = (int32_t)local(col[v][in ? s : std::max<int64_t>(0, n_real[v] - 1)]);
                    *vp++ = in ? value[v][s] : T(0);
                }
        };
        // (threads share the slots evenly, not the blocks: the longest come first)
        const int64_t parts = host_threads(real, (int64_t)out.blocks.size(), 64);
        for_each_item(parts, (int)parts, [&](int64_t part) {
            auto at = std::lower_bound(out.blocks.begin(), out.blocks.end(), slot * part / parts,
                                       [](const GatherBlock &b, int64_t s) { return (int64_t)b.slot_base < s; });
            for (; at != out.blocks.end() && (part + 1 == parts || (int64_t)at->slot_base < slot * (part + 1) / parts); ++at)
                fill_block(*at);
        });
    };
    if (es == 8) fill(double());
    else fill(float());
}

}  // namespace

namespace {

// Second-phase block of one tile (see TileDesc): the fused rows, longest first, cut into units
// of one padded length each.  A unit ends when the next row is shorter and the unit already
// has 64 rows, or when the next row would be padded by more than a quarter.  The padded length
// (stride) is even so that value pairs are aligned; padding entries repeat the row's last
// column with value 0.  local(c) is what the kernel finds the D1 row of column c with.
struct TileBlock {
    std::vector<unsigned char> bytes;
    std::vector<int32_t> rows;      // fused rows in block order
    int32_t n_units = 0, n_entries = 0;
};

template <typename LocalFn>
TileBlock pack_tile(const int32_t *rowptr, const int32_t *colidx, const unsigned char *vals, int es,
                    std::vector<int32_t> list, LocalFn local) {
    auto len = [&](int32_t j) { return (int64_t)rowptr[j + 1] - rowptr[j]; };
    auto align16 = [](size_t x) { return (x + 15) / 16 * 16; };
    TileBlock tb;
    std::stable_sort(list.begin(), list.end(), [&](int32_t a, int32_t b) { return len(a) > len(b); });
    tb.rows = list;
    std::vector<TileUnit> units;
    std::vector<uint16_t> idx;
    std::vector<unsigned char> val;
    const int64_t count = (int64_t)list.size();
    int64_t pos = 0;
    while (pos < count) {
        const int64_t L = len(list[pos]);
        const int64_t stride = (L + 1) / 2 * 2;
        int64_t take = 1;
        while (pos + take < count) {
            const int64_t ln = len(list[pos + take]);
            if (ln == L) {
                ++take;
                continue;
            }
            if (take >= 64 || ln * 4 < L * 3 || ln == 0) break;
            ++take;
        }
        TileUnit u{};
        u.entry_base = (int32_t)idx.size();
        u.row_begin = (int32_t)pos;
        u.n_rows = (int32_t)take;
        u.slots = (int32_t)(stride | (L << 16));
        {
            const size_t at0 = idx.size();
            idx.resize(at0 + (size_t)(take * stride), 0);
            val.resize(idx.size() * es, 0);
            uint16_t *ip = idx.data() + at0;
            unsigned char *vp = val.data() + at0 * es;
            for (int64_t q = pos; q < pos + take; ++q) {
                const int32_t j = list[q];
                const int64_t k0 = rowptr[j], ln = len(j);
                for (int64_t sl = 0; sl < ln; ++sl) *ip++ = (uint16_t)local(colidx[k0 + sl]);
                std::memcpy(vp, vals + (size_t)k0 * es, (size_t)ln * es);
                if (ln > 0)
                    for (int64_t sl = ln; sl < stride; ++sl) *ip++ = (uint16_t)local(colidx[k0 + ln - 1]);
                else
                    ip += stride;
                vp += (size_t)stride * es;
            }
        }
        units.push_back(u);
        pos += take;
    }
    const size_t off_rows2 = align16(units.size() * sizeof(TileUnit));
    const size_t off_idx = align16(off_rows2 + list.size() * 4);
    const size_t off_val = align16(off_idx + idx.size() * 2);
    tb.bytes.assign(align16(off_val + val.size()), 0);
    if (!units.empty()) std::memcpy(tb.bytes.data(), units.data(), units.size() * sizeof(TileUnit));
    if (!list.empty()) std::memcpy(tb.bytes.data() + off_rows2, list.data(), list.size() * 4);
    // operand positions: the even slots of all rows first, then the odd slots, so that the two
    // positions of a pair come from different arrays, by two plain 16-bit reads (one 32-bit read
    // of both would have to be taken apart again by the vector ALU, the scarce unit there)
    uint16_t *ip = reinterpret_cast<uint16_t *>(tb.bytes.data() + off_idx);
    const size_t pairs = idx.size() / 2;
    for (size_t q = 0; q < pairs; ++q) {
        ip[q] = idx[2 * q];
        ip[pairs + q] = idx[2 * q + 1];
    }
    if (!val.empty()) std::memcpy(tb.bytes.data() + off_val, val.data(), val.size());
    tb.n_units = (int32_t)units.size();
    tb.n_entries = (int32_t)idx.size();
    return tb;
}

}  // namespace

// Columns between the rows of a workspace whose rows are shorter than a cache line, ccol or more: rows that straddle
// lines cost a request each time they do, padding makes the array larger.  (R-MAT graphs, fp32, 23 columns, second
// wavefront, us, rows of 92, 96 and 128 bytes: 100000 rows 21.6 / 20.3 / 17.5, 2^20 rows 258 / 240 / 194.)
static int64_t row_pitch(int64_t ccol, int64_t es) {
    const int64_t row = ccol * es;
    auto cost = [&](int64_t pitch) {
        int lines = 0;
        for (int k = 0; k < 32; ++k) lines += (k * pitch % kGatherSliceBytes + row - 1) / kGatherSliceBytes + 1;
        return lines / 32.0 * std::pow((double)pitch / (double)row, 0.4);
    };
    int64_t best = row;
    for (int64_t p = 32; p <= kGatherSliceBytes; p *= 2)
        if (p >= row && p < 2 * row && cost(p) < cost(best)) best = p;
    return best / es;
}

// Share of sampled entries whose column is among those of other sampled ones, as many as an L2 has cache lines
// (Schedule::reuse).  Samples are runs of neighbouring entries, one in each equal part of A.
static double column_reuse(const InspectorInput &in) {
    constexpr int64_t run = 16, lines = ((int64_t)4 << 20) / kGatherSliceBytes;
    if (in.nnz < run) return 1.0;
    std::vector<uint64_t> seen((size_t)(in.n + 63) / 64, 0);
    auto sample = [&](int64_t runs, uint64_t seed, auto f) {
        for (int64_t i = 0; i < runs; ++i) {
            const int64_t lo = in.nnz * i / runs, hi = in.nnz * (i + 1) / runs;
            seed = seed * 6364136223846793005u + 1442695040888963407u;
            const int64_t at = std::min(in.nnz - run, lo + (int64_t)(seed >> 33) % std::max<int64_t>(1, hi - lo));
            for (int64_t e = 0; e < run; ++e) f(in.colidx[at + e]);
        }
    };
    sample(lines / run, 1, [&](int32_t c) { seen[(size_t)c / 64] |= (uint64_t)1 << c % 64; });
    int64_t hits = 0;
    sample(lines / run / 4, 2, [&](int32_t c) { hits += seen[(size_t)c / 64] >> c % 64 & 1; });
    return (double)hits / (double)(lines / 4);
}

// How rows of `sw` columns (of ccol, in column slices) are packed for the gather kernel; `entries` of them in all.
static PackRules pack_rules(const InspectorInput &in, int64_t ccol, int64_t entries, const D1Layout &lay) {
    const int elems = lane_elems(in.dtype, ccol, lay.sw), group = lane_group(lay.sw, elems);
    PackRules r;
    r.nr = 64 / group;
    const int64_t n_cb = (lay.sw + group * elems - 1) / (group * elems);
    r.counts = (int)(lay.n_sl * n_cb);
    // slots that a wave has on average when all blocks are dealt out
    const int64_t waves = (int64_t)std::max(1, in.n_cu) * 4 * gather_waves(in.dtype);
    const int64_t mean = entries / r.nr * lay.n_sl / waves;
    // (rows wider than a wave's load: as much longer, so that the sums of their pieces take no more memory than
    // their entries; below the 16 bits of a block's size)
    r.longest = std::min<int64_t>(32760, std::min<int64_t>(256, std::max<int64_t>(32, round_up(mean / 2, kGatherEntries))) * n_cb);
    return r;
}

tf_status build_schedule(const InspectorInput &in, Schedule &s, std::string &err) {
    const int64_t n = in.n;
    const int es = elem_size(in.dtype);
#ifdef TF_TIMING
    auto tf_tick = std::chrono::steady_clock::now();
#endif
    s = Schedule();
    s.n = n;
    s.nnz = in.nnz;

    // ---- column slice -------------------------------------------------------------------
    const int v = vec_elems(in.dtype);
    int64_t max_cs = in.b_is_sparse ? 64 * v : kMaxMfmaSliceCols;
    // scalar lanes, one column each: the dense kernels at an unaligned width, and the limit of a slice
    // that the caller asks for
    if (in.ccol % v != 0 && (!in.b_is_sparse || in.col_slice > 0 || (in.ccol > max_cs && in.ccol % max_cs < v)))
        max_cs = 64;
    int64_t cs = in.col_slice > 0 ? in.col_slice : in.ccol;
    if (in.col_slice < 0) {
        err = "col_slice must be >= 0";
        return TF_EINVAL;
    }
    cs = std::min<int64_t>(cs, in.ccol);
    if (cs > max_cs) {
        if (in.col_slice > 0) {
            err = "col_slice is wider than the kernels cover for this shape";
            return TF_EUNSUPPORTED;
        }
        cs = max_cs;
    }
    if (in.ccol % v == 0 && cs % v != 0 && cs != in.ccol) {
        err = "col_slice must be a multiple of 16 bytes of elements";
        return TF_EINVAL;
    }
    // ---- fast-memory model --------------------------------------------------------------
    // Per D1 row: the row itself, its id in two buffers (this tile's and the next one's), and an
    // estimate of its share of the second-phase block (row id, packed entries of an average row).
    // The C slice of a dense B takes LDS for good only when the waves read their operands from it.
    const int64_t avg_nnz = n > 0 ? (in.nnz + n - 1) / n : 0;
    s.lds_meta_bytes_per_row = 8 + 4 + avg_nnz * (2 + es);
    const int64_t b_stage = in.b_is_sparse ? lds_sparse_b_bytes_per_row(in.dtype) : 0;
    s.lds_row_granule = lds_row_granule(in.b_is_sparse);
    s.fast_mem_bytes = in.fast_mem_bytes;
    auto model = [&](int64_t width) {
        const bool c_regs = !in.b_is_sparse &&
                            c_in_registers(in.dtype, mfma_blocks((int)width),
                                           mfma_ksteps_special(in.dtype, (int)in.bcol, (int)in.ccol, (int)width));
        s.lds_fixed_bytes =
            (c_regs ? 0 : lds_fixed_bytes(in.dtype, in.b_is_sparse, (int)in.bcol, (int)width)) + 256;
        s.lds_bytes_per_row =
            lds_ldl(in.dtype, in.b_is_sparse, (int)width) * es + s.lds_meta_bytes_per_row + b_stage;
    };
    model(cs);
    // ---- the caller left the tiling to the library ----------------------------------------
    // (no tile size, no tile count, no flag that fixes the kind of tiles).  Then: a quarter of the
    // compute units as the wanted number of tiles (with all of them a small matrix gets tiles of a
    // handful of rows, which fuse nothing); for a dense B whose C operands sit in registers, half
    // of the LDS per tile when that still holds kWantedTileRows rows, so that two workgroups share
    // a compute unit; consecutive or graph-grown tiles, whichever moves fewer bytes; and fused rows
    // that would keep the whole tile machinery alive for next to no work are left to the second
    // wavefront (see below).
    const bool automatic = in.ct_size == 0 && in.p == 0 &&
                           !(in.flags & (TF_FLAG_REORDER | TF_FLAG_NO_SPLIT));
    s.automatic = automatic;
    if (automatic && !in.b_is_sparse && in.fast_mem_bytes >= 128 * 1024) {
        const bool c_regs = c_in_registers(in.dtype, mfma_blocks((int)cs),
                                           mfma_ksteps_special(in.dtype, (int)in.bcol, (int)in.ccol, (int)cs));
        const int64_t half = in.fast_mem_bytes / 2;
        if (c_regs && s.lds_fixed_bytes + kWantedTileRows * s.lds_bytes_per_row <= half)
            s.fast_mem_bytes = half;
    }
    // ---- step 1: tile size --------------------------------------------------------------
    const int64_t ct = in.ct_size > 0 ? in.ct_size : 2048;
    const int64_t p = in.p > 0 ? in.p : (automatic ? std::max(1, in.n_cu / 4) : 32);
    int64_t t = ct;
    if (n > 0 && (n + ct - 1) / ct < p) t = (n + p - 1) / p;
    if (t < 1) t = 1;
    s.t = (int32_t)std::min<int64_t>(t, INT32_MAX);

    // A default slice is narrowed (cCol / 2, / 4, ... rounded up to 16 columns; thirds leave a
    // ragged last slice and measured worse than either neighbour) until the fast
    // memory holds a tile of t rows, or of kWantedTileRows if t is larger: a C slice that fills
    // the LDS leaves tiles of a few rows, which fuse nothing.  If no width gets there the one
    // with the most rows is taken.  A slice the caller asked for is taken as given.
    if (in.col_slice == 0) {
        auto capacity = [&]() -> int64_t {
            const int64_t room = s.fast_mem_bytes - s.lds_fixed_bytes;
            if (room < s.lds_bytes_per_row) return 0;
            return room / s.lds_bytes_per_row / s.lds_row_granule * s.lds_row_granule;
        };
        const int64_t want = round_up(std::min<int64_t>(std::max<int64_t>(t, 1), kWantedTileRows),
                                      s.lds_row_granule);
        const int64_t widest = cs;
        int64_t best_cs = cs, best_rows = capacity();
        for (int64_t k = 2; best_rows < want && cs > 16; k *= 2) {
            const int64_t c = round_up((widest + k - 1) / k, 16);
            // (more than 64 scalar lanes are not covered)
            if (c >= cs || (in.b_is_sparse && c > 64 && lane_elems(in.dtype, in.ccol, c) == 1)) continue;
            cs = c;
            model(cs);
            if (capacity() > best_rows) {
                best_rows = capacity();
                best_cs = cs;
            }
        }
        cs = best_cs;
        model(cs);
    }
    if (tile_footprint(s, 1) > s.fast_mem_bytes) {
        err = "fast_mem_bytes cannot hold one D1 row of the chosen column slice (plus the C slice)";
        return TF_EUNSUPPORTED;
    }
    s.col_slice = (int32_t)cs;
    s.n_slices = (int32_t)((in.ccol + cs - 1) / cs);

    // ---- tiles: lists of first-operation rows -------------------------------------------
    // first_rows holds the rows tile after tile; tile_first_ptr delimits the tiles.
    const bool allow_split = !(in.flags & TF_FLAG_NO_SPLIT);
    struct Tiling {
        std::vector<int32_t> first_rows, tile_first_ptr;
        int64_t n_coarse = 0;
        bool grown = false;
    };
    auto make_grown = [&](Tiling &tl) {
        // Tiles grown along the dependence graph: as many rows as fit the fast memory (and at
        // most t), collected breadth first from the lowest row not yet in a tile by following
        // each row's column indices; when a search runs dry the tile goes on from the next
        // free row.  Rows inside a tile are kept in ascending order.
        tl.grown = true;
        tl.first_rows.resize((size_t)n);
        tl.tile_first_ptr.assign(1, 0);
        int64_t cap = std::min<int64_t>(automatic ? 65536 : t, 65536);
        while (cap > 1 && tile_footprint(s, cap) > s.fast_mem_bytes) --cap;
        cap = std::max<int64_t>(1, cap / s.lds_row_granule * s.lds_row_granule);
        if (tile_footprint(s, cap) > s.fast_mem_bytes) cap = 1;
        // One workgroup per compute unit walks the tiles of its column slice, so a tile count that
        // is not a multiple of the workgroups per slice leaves most of them waiting for the few
        // that got one tile more (304 tiles on 256 units: two rounds for the work of 1.2).  The
        // tiles are made smaller (by less than half) so that the count becomes such a multiple.
        // With fewer tiles than workgroups there is nothing to balance.
        if (n > 0 && in.n_cu > 0) {
            const int64_t per_slice = std::max<int64_t>(1, in.n_cu / s.n_slices);
            const int64_t count0 = (n + cap - 1) / cap;
            if (count0 >= per_slice) {
                const int64_t count = round_up(count0, per_slice);
                const int64_t even = round_up((n + count - 1) / count, s.lds_row_granule);
                if (even >= 1 && even < cap) cap = even;
            }
        }
        // (Growing the tiles of several row ranges at once on the host threads was measured: tiles
        // cut off at the end of a range fuse less -- 80.6 % of config 2's rows with four ranges, 74 %
        // with ranges of one tile height, against 82 % -- which costs every execution more than the
        // millisecond of inspector time it saves.)
        // tile_no[row]: number of the row's tile, -1 while the row is free
        std::vector<int32_t> tile_no((size_t)n, -1), queue;
        queue.reserve((size_t)cap);
        int64_t seed = 0, filled = 0;
        int32_t vt = 0;
        while (filled < n) {
            queue.clear();
            size_t head = 0;
            while ((int64_t)queue.size() < cap && filled + (int64_t)queue.size() < n) {
                if (head == queue.size()) {               // start (or restart) from a free row
                    while (tile_no[seed] >= 0) ++seed;
                    tile_no[seed] = vt;
                    queue.push_back((int32_t)seed);
                    continue;
                }
                const int32_t j = queue[head++];
                for (int64_t q = in.rowptr[j]; q < in.rowptr[j + 1]; ++q) {
                    const int32_t c = in.colidx[q];
                    if (tile_no[c] < 0 && (int64_t)queue.size() < cap) {
                        tile_no[c] = vt;
                        queue.push_back(c);
                    }
                }
            }
            filled += (int64_t)queue.size();
            tl.tile_first_ptr.push_back((int32_t)filled);
            ++vt;
        }
        // the rows of every tile in ascending order: one pass over the rows instead of a sort per tile
        std::vector<int32_t> cursor(tl.tile_first_ptr.begin(), tl.tile_first_ptr.end() - 1);
        for (int64_t row = 0; row < n; ++row)
            tl.first_rows[(size_t)cursor[(size_t)tile_no[(size_t)row]]++] = (int32_t)row;
        tl.n_coarse = (int64_t)tl.tile_first_ptr.size() - 1;
    };
    auto make_consecutive = [&](Tiling &tl) {
        // Algorithm 1: uniform tiles of t consecutive rows (step 1), halved until they fit (step 2)
        tl.first_rows.resize((size_t)n);
        tl.tile_first_ptr.assign(1, 0);
        std::vector<Range> tiles;
        for (int64_t i0 = 0; i0 < n; i0 += t) {
            ++tl.n_coarse;
            split_tile(s, Range{i0, std::min(n, i0 + t)}, allow_split, tiles);
        }
        std::iota(tl.first_rows.begin(), tl.first_rows.end(), 0);
        for (const Range &r : tiles) tl.tile_first_ptr.push_back((int32_t)r.i1);
    };
    // What a tiling is worth, without packing anything: the stored entries of the rows it fuses
    // (all of them, and those of rows that are not direct rows) and the number of D1 rows it spills.
    struct Worth {
        int64_t fused_nnz = 0, lds_nnz = 0, lds_rows = 0, spill_rows = 0;
        std::vector<uint8_t> spilled;      // the spill set of the tiling (before any row is demoted)
    };
    auto evaluate = [&](const Tiling &tl) {
        const int64_t ntl = (int64_t)tl.tile_first_ptr.size() - 1;
        std::vector<int32_t> tile_of((size_t)n);
        for (int64_t vt = 0; vt < ntl; ++vt)
            for (int64_t q = tl.tile_first_ptr[vt]; q < tl.tile_first_ptr[vt + 1]; ++q)
                tile_of[tl.first_rows[q]] = (int32_t)vt;
        std::vector<uint8_t> spilled((size_t)n, 0);
        std::vector<Worth> part((size_t)ntl);
        for_each_item(ntl, host_threads(in.nnz, ntl, 16), [&](int64_t vt) {
            Worth &w = part[(size_t)vt];
            for (int64_t fq = tl.tile_first_ptr[vt]; fq < tl.tile_first_ptr[vt + 1]; ++fq) {
                const int64_t j = tl.first_rows[fq];
                const int64_t k0 = in.rowptr[j], k1 = in.rowptr[j + 1];
                bool inside = k1 - k0 < 32768;
                for (int64_t q = k0; inside && q < k1; ++q) inside = tile_of[in.colidx[q]] == (int32_t)vt;
                if (inside) {
                    w.fused_nnz += k1 - k0;
                    if (!(k1 == k0 || (k1 - k0 == 1 && in.colidx[k0] == (int32_t)j))) {
                        w.lds_nnz += k1 - k0;
                        ++w.lds_rows;
                    }
                } else {
                    for (int64_t q = k0; q < k1; ++q) {
                        uint8_t *m = &spilled[(size_t)in.colidx[q]];
                        if (!__atomic_load_n(m, __ATOMIC_RELAXED)) __atomic_store_n(m, (uint8_t)1, __ATOMIC_RELAXED);
                    }
                }
            }
        });
        Worth w;
        for (const Worth &pw : part) {
            w.fused_nnz += pw.fused_nnz;
            w.lds_nnz += pw.lds_nnz;
            w.lds_rows += pw.lds_rows;
        }
        w.spill_rows = std::accumulate(spilled.begin(), spilled.end(), (int64_t)0);
        w.spilled = std::move(spilled);
        return w;
    };
    // Rows that reach far (graphs): mean distance, over a sample of the entries, between a row and
    // the columns it holds, in bytes of D1 rows, against the 4 MiB of one XCD's L2.
    bool far_rows = false;
    if (n > 0 && in.nnz > 0) {
        // the sample: 64 runs of up to 1024 consecutive rows, evenly spread (runs, not single rows:
        // their entries are read as a stream)
        const int64_t run = std::min<int64_t>(1024, std::max<int64_t>(1, n / 64));
        const double far_b = 1048576.0 / ((double)in.bcol * es);       // rows of B in 1 MiB
        double dist = 0.0;
        int64_t cnt = 0, far = 0;
        for (int64_t k = 0; k < 64; ++k) {
            const int64_t j0 = std::min(n - run, n * k / 64);
            for (int64_t j = j0; j < j0 + run; ++j)
                for (int64_t q = in.rowptr[j]; q < in.rowptr[j + 1]; ++q) {
                    const double d = std::abs((double)in.colidx[q] - (double)j);
                    dist += d;
                    far += d > far_b;
                    ++cnt;
                }
        }
        far_rows = cnt > 0 && dist / (double)cnt * (double)in.ccol * es > 4.0 * 1048576.0;
        s.far_b_share = cnt > 0 ? (double)far / (double)cnt : 0.0;
    }
    s.far_rows = far_rows;
    if (far_rows) s.reuse = column_reuse(in);
    bool demote_lds_rows = false;
    std::vector<uint8_t> known_spill;      // spill set of the chosen tiling, when it was evaluated
    Tiling tiling;
    TF_TICK("setup, far-row sample");
    if (in.flags & TF_FLAG_REORDER) {
        make_grown(tiling);
        TF_TICK("grown tiles");
    } else {
        make_consecutive(tiling);
        if (automatic && in.nnz > 0) {
            Worth w = evaluate(tiling);
            TF_TICK("consecutive tiles + worth");
            // consecutive tiles that fuse less than half of the work of a matrix whose rows stay
            // near the diagonal (a stencil in natural ordering): try tiles grown along the graph
            // and keep them if they spill fewer D1 rows, i.e. move fewer bytes
            if (!far_rows && 2 * w.fused_nnz < in.nnz) {
                Tiling grown;
                make_grown(grown);
                TF_TICK("grown tiles");
                Worth wg = evaluate(grown);
                TF_TICK("worth of grown tiles");
                if (wg.spill_rows < w.spill_rows) {
                    tiling = std::move(grown);
                    w = std::move(wg);
                }
            }
            // Fused rows that read the LDS tile make every workgroup keep a tile in LDS and pass
            // two barriers per tile.  When they hold under 2 % of the entries that machinery costs
            // more than the D1 round trip it saves (measured on the graph configurations: a
            // handful of such rows, first wavefront 0.44 ms with tiles against 0.31 ms without):
            // they are left to the second wavefront and the first wavefront streams.
            demote_lds_rows = w.lds_rows > 0 && 50 * w.lds_nnz < in.nnz;
            known_spill = std::move(w.spilled);
        }
    }
    s.first_rows = std::move(tiling.first_rows);
    s.tile_first_ptr = std::move(tiling.tile_first_ptr);
    s.n_coarse_tiles = tiling.n_coarse;
    s.grown_tiles = tiling.grown;
    const int64_t nt = (int64_t)s.tile_first_ptr.size() - 1;
    for (int64_t vt = 0; vt < nt; ++vt) {
        const int64_t rows = s.tile_first_ptr[vt + 1] - s.tile_first_ptr[vt];
        if (tile_footprint(s, rows) > s.fast_mem_bytes) {
            err = "a tile does not fit the fast memory and splitting is disabled";
            return TF_EUNSUPPORTED;
        }
        s.max_tile_rows = std::max(s.max_tile_rows, rows);
    }

    // ---- classification: a row is fused when every column it refers to is produced by the
    // tile that produces its own row; fused rows are packed with tile-local column indices ----
    s.tile_second_ptr.resize(nt + 1);
    s.spill.assign((size_t)n, 0);
    const unsigned char *vals = static_cast<const unsigned char *>(in.vals);
    std::vector<TileBlock> blocks((size_t)nt);
    // the packed entries of a tile name their D1 operand by its position in the LDS tile, in units of
    // 16 bytes (16 bits: enough for 1 MiB of tile)
    const int32_t pitch16 = (int32_t)(lds_ldl(in.dtype, in.b_is_sparse, (int)cs) * es / 16);
    if (s.max_tile_rows * pitch16 > 65536) {
        err = "a tile is larger than 1 MiB (tile-local operand offsets are 16 bit)";
        return TF_EUNSUPPORTED;
    }
    std::vector<int32_t> wf1;
    int64_t lds_nonempty = 0;          // fused rows that read the LDS tile and have entries
    // A row belongs to one tile: there it is a candidate for fusion and there its D1 row is
    // produced.  With TF_FLAG_SKIP_UNREAD the D1 rows that no row of A reads are not produced at
    // all: they leave the tiles' first lists (a tile keeps at least one row) and get no place in LDS.
    // (member_*: the tiles' rows before any are taken out; the lists themselves when none are)
    const bool skip_rows = (in.flags & TF_FLAG_SKIP_UNREAD) != 0;
    std::vector<int32_t> all_ptr, all_rows;
    if (skip_rows) {
        all_ptr = s.tile_first_ptr;
        all_rows = s.first_rows;
    }
    const std::vector<int32_t> &member_ptr = skip_rows ? all_ptr : s.tile_first_ptr;
    const std::vector<int32_t> &member_rows = skip_rows ? all_rows : s.first_rows;
    if (skip_rows) {
        std::vector<uint8_t> read((size_t)n, 0);
        for (int64_t q = 0; q < in.nnz; ++q) read[in.colidx[q]] = 1;
        int64_t kept = 0;
        s.max_tile_rows = 0;
        for (int64_t vt = 0; vt < nt; ++vt) {
            const int64_t before = kept;
            for (int64_t q = member_ptr[vt]; q < member_ptr[vt + 1]; ++q)
                if (read[member_rows[q]]) s.first_rows[kept++] = member_rows[q];
            if (kept == before && member_ptr[vt + 1] > member_ptr[vt])
                s.first_rows[kept++] = member_rows[member_ptr[vt]];
            s.tile_first_ptr[vt + 1] = (int32_t)kept;
            s.max_tile_rows = std::max(s.max_tile_rows, kept - before);
        }
        s.first_rows.resize((size_t)kept);
    }
    std::vector<int32_t> tile_of((size_t)n), local_of((size_t)n, 0);
    // kept[row]: the tile produces the D1 row (always, unless unread rows are skipped);
    // direct_kind[row]: 1 = the row of D is the D1 row times its only entry, the diagonal one;
    // 2 = the row of D is empty; both leave from the registers that hold the D1 row
    std::vector<uint8_t> kept((size_t)n, 0), direct_kind((size_t)n, 0);
    // (every row is in one tile: the threads write to places of their own tiles only)
    for_each_item(nt, host_threads(in.nnz, nt, 16), [&](int64_t vt) {
        for (int64_t q = member_ptr[vt]; q < member_ptr[vt + 1]; ++q)
            tile_of[member_rows[q]] = (int32_t)vt;
        for (int64_t q = s.tile_first_ptr[vt]; q < s.tile_first_ptr[vt + 1]; ++q) {
            local_of[s.first_rows[q]] = (int32_t)(q - s.tile_first_ptr[vt]);
            kept[s.first_rows[q]] = 1;
        }
    });
    std::vector<int32_t> seen((size_t)n, -1);      // Eq. 2: distinct columns per tile
    // Per tile: which of its rows are fused, and their packed block.  Tiles are independent (a fused
    // row only names columns of its own tile, so even `seen` is written at disjoint places), which
    // lets several host threads share the tiles of a large matrix; the results are put together
    // in tile order afterwards, so the schedule does not depend on the number of threads.
    struct TileResult {
        std::vector<int32_t> wf1, direct, demoted_rows;
        int64_t tile_nnz = 0, uc = 0, nj = 0, demoted = 0, lds_nonempty = 0;
    };
    std::vector<TileResult> res((size_t)nt);
    auto classify = [&](int64_t vt) {
        TileResult &tr = res[(size_t)vt];
        std::vector<int32_t> tile_rows;
        for (int64_t fq = member_ptr[vt]; fq < member_ptr[vt + 1]; ++fq) {
            const int64_t j = member_rows[fq];
            // (a row of 32768 entries or more, possible only with duplicates, is left to the second
            // wavefront: the tile units store lengths in 15 bits)
            bool inside = in.rowptr[j + 1] - in.rowptr[j] < 32768;
            for (int64_t q = in.rowptr[j]; inside && q < in.rowptr[j + 1]; ++q) {
                if (tile_of[in.colidx[q]] != (int32_t)vt) {
                    inside = false;
                    break;
                }
            }
            const int64_t ln = in.rowptr[j + 1] - in.rowptr[j];
            const bool direct = kept[j] && (ln == 0 || (ln == 1 && in.colidx[in.rowptr[j]] == (int32_t)j));
            if (inside && demote_lds_rows && !direct && ln > 0) {       // (a row without entries reads no tile)
                inside = false;
                ++tr.demoted;
                tr.demoted_rows.push_back((int32_t)j);
            }
            if (inside) {
                if (direct) {
                    direct_kind[j] = ln == 0 ? 2 : 1;
                    tr.direct.push_back((int32_t)j);
                } else {
                    tile_rows.push_back((int32_t)j);
                    direct_kind[j] = 3;          // fused through the LDS tile
                    if (ln > 0) ++tr.lds_nonempty;
                }
                for (int64_t q = in.rowptr[j]; q < in.rowptr[j + 1]; ++q) {
                    const int32_t c = in.colidx[q];
                    if (seen[c] != (int32_t)vt) {
                        seen[c] = (int32_t)vt;
                        ++tr.uc;
                    }
                }
                tr.tile_nnz += in.rowptr[j + 1] - in.rowptr[j];
            } else {
                tr.wf1.push_back((int32_t)j);
            }
        }
        tr.nj = (int64_t)(tile_rows.size() + tr.direct.size());
        blocks[(size_t)vt] = pack_tile(in.rowptr, in.colidx, vals, es, tile_rows,
                                       [&](int32_t c) { return local_of[c] * pitch16; });
    };
    TF_TICK("tile maps");
    for_each_item(nt, host_threads(in.nnz, nt, 16), classify);
    TF_TICK("classify + pack tiles");
    for (int64_t vt = 0; vt < nt; ++vt) {
        const TileResult &tr = res[(size_t)vt];
        const int64_t rows = s.tile_first_ptr[vt + 1] - s.tile_first_ptr[vt];
        wf1.insert(wf1.end(), tr.wf1.begin(), tr.wf1.end());
        s.tile_second_ptr[vt] = (int32_t)s.second_rows.size();
        s.second_rows.insert(s.second_rows.end(), blocks[(size_t)vt].rows.begin(),
                             blocks[(size_t)vt].rows.end());
        s.second_rows.insert(s.second_rows.end(), tr.direct.begin(), tr.direct.end());
        s.n_demoted_rows += tr.demoted;
        lds_nonempty += tr.lds_nonempty;
        s.n_lds_rows += (int64_t)blocks[(size_t)vt].rows.size();
        s.n_direct_rows += (int64_t)tr.direct.size();
        // Eq. 2 (diagnostic): (nz + uc + t + |J|) * cCol + idx, counted in elements; for a dense B
        // the tile's rows x bCol block of B is added to nz, a sparse B is unknown here.
        const double nz = (double)tr.tile_nnz + (in.b_is_sparse ? 0.0 : (double)rows * in.bcol);
        const double idx = (double)(rows + 1) + (double)tr.tile_nnz;
        s.eq2_cost_max = std::max(s.eq2_cost_max, (nz + tr.uc + rows + tr.nj) * (double)in.ccol + idx);
        s.fused_nnz += tr.tile_nnz;
    }
    s.tile_second_ptr[nt] = (int32_t)s.second_rows.size();
    s.n_fused_rows = (int64_t)s.second_rows.size();
    if (!s.grown_tiles && !std::is_sorted(wf1.begin(), wf1.end())) std::sort(wf1.begin(), wf1.end());

    TF_TICK("collect tiles");
    // ---- spill set ----------------------------------------------------------------------
    if (!known_spill.empty() && !(in.flags & TF_FLAG_SKIP_UNREAD)) {
        // the tiling was evaluated: its spill set is known; rows left to the second wavefront since
        // then add the rows they read
        s.spill = std::move(known_spill);
        for (const TileResult &tr : res)
            for (int32_t j : tr.demoted_rows)
                for (int64_t q = in.rowptr[j]; q < in.rowptr[j + 1]; ++q) s.spill[(size_t)in.colidx[q]] = 1;
    } else {
        // (several threads may mark the same row: every one of them stores the same byte)
        for_each_item((int64_t)wf1.size(), host_threads(in.nnz, (int64_t)wf1.size(), 4096), [&](int64_t k) {
            const int32_t j = wf1[(size_t)k];
            for (int64_t q = in.rowptr[j]; q < in.rowptr[j + 1]; ++q) {
                // (a marked row is not written again: the columns of hub rows would otherwise keep
                // their cache lines travelling between the threads)
                uint8_t *m = &s.spill[(size_t)in.colidx[q]];
                if (!__atomic_load_n(m, __ATOMIC_RELAXED)) __atomic_store_n(m, (uint8_t)1, __ATOMIC_RELAXED);
            }
        });
    }
    s.n_spill_rows = std::accumulate(s.spill.begin(), s.spill.end(), (int64_t)0);
    if (s.n_spill_rows > (int64_t)kInfoSlotMask) {
        err = "more than 2^28 D1 rows cross tiles";
        return TF_EUNSUPPORTED;
    }
    // Only the rows in the spill set reach device memory (one barrier: nothing else crosses tiles),
    // so the workspace has one slot per such row, in row order.
    s.spill_slot.assign((size_t)n, -1);
    {
        int32_t slot = 0;
        for (int64_t i = 0; i < n; ++i)
            if (s.spill[(size_t)i]) s.spill_slot[(size_t)i] = slot++;
    }
    // ---- layout of the workspace = column slices of the gather kernel ---------------------
    // On a matrix whose rows reach far (a graph) every XCD's L2 sees the same hot rows of D1 and
    // holds them all, whole: the eight caches together are worth one.  With n_sl slices each XCD
    // gathers sw-wide pieces of the rows, so the hot set is spread over the caches, at the price of
    // reading the packed entries of A once per slice.  Slices of one cache line each, up to eight (R-MAT graphs,
    // second wavefront, us, whole rows / slices of two lines / of one: 30000 rows fp32 128 columns 23.1 / 17.9 /
    // 17.0; 100000 rows fp64 64 columns 63.9 / 56.3 / 55.8, fp32 64 columns 30.0 / - / 28.6; 300000 rows fp64 128
    // columns 574 / 476 (two slices) / 373 (eight); 2^20 rows fp32 128 columns 930 / 837 / 703; of half a line,
    // 2^20 rows, 1111).  Matrices whose rows stay near the diagonal (stencils, bands) keep one slice.
    {
        int n_sl = 1;
        int64_t sw = in.ccol;
        auto usable = [&](int k) {
            if (k == 1) return true;
            if (in.ccol % v || in.ccol % k) return false;
            // (the MFMA phase stores 16-column blocks that start at multiples of the fused column
            // slice: they must not straddle a slice of the workspace)
            if (s.n_slices > 1 && cs % 16 != 0) return false;
            const int64_t sw = in.ccol / k;
            return sw % 16 == 0 && (sw & (sw - 1)) == 0 && sw * es >= 64;
        };
        s.d1.rows = std::max<int64_t>(1, s.n_spill_rows);
        if (in.gather_slices > 0) {
            if ((in.gather_slices != 1 && in.gather_slices != 2 && in.gather_slices != 4 &&
                 in.gather_slices != 8) || !usable(in.gather_slices)) {
                err = "gather_slices must be 1, 2, 4 or 8 and leave slices of a power of two of columns, "
                      "at least 16 and at least 64 bytes";
                return TF_EINVAL;
            }
            n_sl = in.gather_slices;
            sw = in.ccol / n_sl;
        } else if (!wf1.empty() && far_rows) {
            if (in.ccol * es > kGatherSliceBytes) {
                int64_t w = kGatherSliceBytes / es;
                while (w * kXcds < in.ccol) w *= 2;
                // (the last slice may be narrower in use, down to one lane's 16 bytes)
                const int64_t k = (in.ccol + w - 1) / w;
                if ((in.ccol - 1) % w + 1 >= v && (s.n_slices == 1 || cs % 16 == 0) &&
                    line_slices_pay(k * w * es, in.ccol * es, s.reuse)) {
                    sw = w;
                    n_sl = (int)k;
                }
            } else {
                sw = row_pitch(in.ccol, es);
            }
            // (the entry point with the library's own workspace takes what it took)
            const int64_t bytes = s.d1.rows * es;
            if (!in.b_is_sparse && bytes * n_sl * sw > kStaticScratchBytes && bytes * in.ccol <= kStaticScratchBytes) {
                n_sl = 1;
                sw = in.ccol;
            }
        }
        s.d1.n_sl = n_sl;
        s.d1.sw = (int32_t)sw;
    }
    TF_TICK("spill set, slots, layout");
    // ---- per-tile blocks (see TileDesc) ---------------------------------------------------
    s.tile_desc.resize((size_t)nt);
    s.first_stride = (int32_t)round_up(std::max<int64_t>(s.max_tile_rows, 1), 16);
    s.tile_first.assign((size_t)nt * s.first_stride, 0);
    s.tile_info.assign((size_t)nt * s.first_stride, 0u);
    if (s.n_direct_rows > 0) {
        s.tile_scale.resize((size_t)nt * s.first_stride * es);
        std::memset(s.tile_scale.data(), 0, s.tile_scale.size());
    }
    {
        int64_t total = 0;
        for (int64_t vt = 0; vt < nt; ++vt) {
            s.tile_desc[(size_t)vt].meta_off = total;
            total += (int64_t)blocks[(size_t)vt].bytes.size();
            s.second_block_cap = std::max<int64_t>(s.second_block_cap, (int64_t)blocks[(size_t)vt].bytes.size());
        }
        s.tile_meta_bytes = (size_t)total + 64;           // the kernels may read one piece past an empty block
        s.tile_meta.reset(new unsigned char[s.tile_meta_bytes]);
        std::memset(s.tile_meta.get() + total, 0, 64);
    }
    for_each_item(nt, host_threads(in.nnz, nt, 16), [&](int64_t vt) {
        const int64_t f0 = s.tile_first_ptr[vt], f1 = s.tile_first_ptr[vt + 1];
        TileBlock &tb = blocks[(size_t)vt];
        TileDesc &d = s.tile_desc[(size_t)vt];
        d.n_rows = (int32_t)(f1 - f0);
        d.n_units = tb.n_units;
        d.n_second = (int32_t)tb.rows.size();
        d.n_entries = tb.n_entries;
        d.s_bytes = (int32_t)tb.bytes.size();
        d.reserved = 0;
        int32_t *first = s.tile_first.data() + (size_t)vt * s.first_stride;
        uint32_t *info = s.tile_info.data() + (size_t)vt * s.first_stride;
        for (int64_t q = f0; q < f1; ++q) {
            const int32_t row = s.first_rows[q];
            first[q - f0] = row;
            uint32_t w = s.spill[row] ? (kInfoSpill | (uint32_t)s.spill_slot[row]) : 0u;
            if (direct_kind[row] == 1) {
                w |= kInfoDirect;
                std::memcpy(s.tile_scale.data() + ((size_t)vt * s.first_stride + (size_t)(q - f0)) * es,
                            vals + (size_t)in.rowptr[row] * es, (size_t)es);
            } else if (direct_kind[row] == 2) {
                w |= kInfoZero;
            }
            info[q - f0] = w;
        }
        // (padding repeats the last row, with an empty info word)
        for (int64_t q = f1 - f0; q < s.first_stride; ++q) first[q] = s.first_rows[f1 - 1];
        if (!tb.bytes.empty()) std::memcpy(s.tile_meta.get() + d.meta_off, tb.bytes.data(), tb.bytes.size());
        TileBlock().bytes.swap(tb.bytes);
    });
    // A plan none of whose fused rows reads the LDS tile needs no tiles at execution: the first
    // wavefront streams through the rows, and what happens to each finished D1 row is told by a word
    // per row.  (Fused rows without entries read nothing: where unread D1 rows are skipped some of
    // them have no D1 row of their own to leave with and sit in the tiles' second lists; by row they
    // are zero rows like the others.)  With TF_FLAG_SKIP_UNREAD only a CSR B streams: its kernel
    // leaves out single rows (kInfoSkip), the dense product works on blocks of sixteen.
    const bool skip_unread = in.flags & TF_FLAG_SKIP_UNREAD;
    s.streaming = n > 0 && lds_nonempty == 0 && (!skip_unread || in.b_is_sparse);
    if (s.streaming) {
        s.row_info.assign((size_t)n, 0u);
        const bool scales = s.n_direct_rows > 0;
        if (scales) {
            s.row_scale.resize((size_t)n * es);
            std::memset(s.row_scale.data(), 0, s.row_scale.size());
        }
        for_each_item(nt, host_threads(in.nnz, nt, 16), [&](int64_t vt) {
            for (int64_t q = member_ptr[vt]; q < member_ptr[vt + 1]; ++q) {
                const int32_t row = member_rows[q];
                uint32_t w = s.spill[row] ? (kInfoSpill | (uint32_t)s.spill_slot[row]) : 0u;
                if (direct_kind[row] == 1) {
                    w |= kInfoDirect;
                    std::memcpy(s.row_scale.data() + (size_t)row * es, vals + (size_t)in.rowptr[row] * es, (size_t)es);
                } else if (direct_kind[row] == 2 || direct_kind[row] == 3) {
                    w |= kInfoZero;
                }
                if (skip_unread && !kept[row]) w |= kInfoSkip;
                s.row_info[(size_t)row] = w;
            }
        });
    }
    {
        // LDS actually needed with the second-phase blocks staged: everything but the estimate
        const int64_t rows_cap = round_up(s.max_tile_rows, s.lds_row_granule);
        const int64_t need = s.lds_fixed_bytes + s.second_block_cap +
                             rows_cap * (s.lds_bytes_per_row - s.lds_meta_bytes_per_row + 8);
        s.second_block_in_lds = need <= s.fast_mem_bytes;
    }

    TF_TICK("tile blocks, row arrays");
    // ---- balance: blocks of the second wavefront -------------------------------------------
    int64_t wf1_nnz = 0;
    for (int32_t j : wf1) wf1_nnz += in.rowptr[j + 1] - in.rowptr[j];
    auto slot_of = [&](int32_t c) { return s.spill_slot[(size_t)c]; };
    pack_rows(in.rowptr, in.colidx, vals, es, std::move(wf1), pack_rules(in, in.ccol, wf1_nnz, s.d1), slot_of, s.wf1);
    s.wf1_rows = s.wf1.rows;
    s.wf1_unit_ptr.clear();
    // (a row that is cut over several blocks is one unit there)
    for (size_t k = 0; k < s.wf1.blocks.size(); ++k)
        if (s.wf1.blocks[k].info >> 6 && (k >= s.wf1.cuts.size() || s.wf1.cuts[k].skip == 0))
            s.wf1_unit_ptr.push_back(s.wf1.blocks[k].row_begin);
    if (!std::is_sorted(s.wf1_unit_ptr.begin(), s.wf1_unit_ptr.end())) std::sort(s.wf1_unit_ptr.begin(), s.wf1_unit_ptr.end());
    s.wf1_unit_ptr.push_back((int32_t)s.wf1_rows.size());
    TF_TICK("second-wavefront units");
    return TF_OK;
}

// Estimated microseconds of the fused calls on a matrix whose rows stay near the diagonal, in two
// wavefronts and in one pass.  The rates (bytes per microsecond) are fits to measured executions.
// Tiles in LDS: the kernels move B and D at 3.2 TB/s.  Unaligned widths take them 1.1 to 1.5 times as long
// (the middle half of 2206 bands and 2D and 3D stencils of 3000 to 3 million rows, 4 to 128 columns: 0.9 to
// 1.7 times); they are charged three times, with which the rule takes the slower way by more than 5 % on 33
// of these plans, by 1.56 times at most.  (1.25 times and 25 us for fp64: 12 of them, but ten plans lose up
// to a fifth that have the right way now.)
static double two_wavefronts_us(const InspectorInput &in) {
    const double es = elem_size(in.dtype), n = (double)in.n, nnz = (double)in.nnz;
    const int v = vec_elems(in.dtype);
    const double aligned = in.bcol % v || in.ccol % v ? 3.0 : 1.0;
    return 15.0 + aligned * (n * (in.bcol + 2.0 * in.ccol) * es / 3.2e6 + nnz * in.ccol * es / 25e6);
}
// Matrix instructions of one block of the kernel, back to back.
static double block_mfma_us(const InspectorInput &in, int ks) {
    return ks * vec_elems(in.dtype) * ((in.ccol + 15) / 16) * (in.dtype == TF_F64 ? 64 : 32) / 2400.0;
}
// A first wavefront without tiles: both kernels take rows of any alignment in 16-byte pieces.  The
// product's waves start and end with a block's multiplications, the gather gets 10 TB/s (lognormal rows of
// mean length 10 and 18, and R-MAT graphs; estimate / measured: 200000 rows fp32 64 -> 64 114 / 99 and 159 /
// 145 us, fp64 128 -> 128 427 / 442 and 600 / 642, 50000 rows fp32 32 -> 32 25 / 26, 50 -> 23 26 / 28, R-MAT of
// 4000 rows fp32 50 -> 23 13 / 14, 128 -> 128 23 / 28, fp64 64 -> 64 19 / 23).
static double streaming_wavefronts_us(const InspectorInput &in, int ks) {
    const double es = elem_size(in.dtype), n = (double)in.n, nnz = (double)in.nnz;
    return 11.0 + 2.0 * block_mfma_us(in, ks) + n * (in.bcol + 2.0 * in.ccol) * es / 3.2e6 + nnz * in.ccol * es / 10e6;
}
// The one-pass kernel gathers rows of B out of the L2 at 18 TB/s and streams at 5 TB/s.  `entries`: with
// padding, where that is known; `far`: the share of them whose row of B is not in the L2.
static double one_pass_us(const InspectorInput &in, double entries, double far = 0.0) {
    const double es = elem_size(in.dtype), n = (double)in.n;
    return 5.0 + entries * in.bcol * es * (1.0 / 18e6 + far / 32e6) + n * (in.bcol + in.ccol) * es / 5e6;
}
// What rows of unequal length add to it: the multiplications of blocks that hold fewer rows than `per_block`,
// and what the wave with the most passes of gathers takes longer than it would with blocks of mean length.  A
// pass waits for its gathers, 0.8 us (band of 20011 rows, eight of them of 400 and of 1024 entries, uncut: fp32
// 32 columns 48 and 116 us, 64 columns 66 and 165, fp64 128 columns 135 and 374: 0.87, 0.79 and 0.77 us a
// pass).  Blocks are dealt to the waves of an XCD as k_gather_gemm takes them in whole rounds; that a short last
// round of wide rows is spread over the workgroups there is left out.  That some waves have a block more than
// others is no matter of row lengths, and in the fits of one_pass_us already (band of 50000 rows of 41, fp64 100 ->
// 100, where it was charged here too: 169 us in two wavefronts, 121 in one pass).
static double one_pass_tail_us(const InspectorInput &in, const ChainPack &c, int ks, int64_t per_block) {
    const int em = chain_entries(in.dtype, ks, c.early);
    const int64_t nb = (int64_t)c.blocks.size(), per = (nb + kXcds - 1) / kXcds;
    const int per_simd = chain_waves(in.dtype, ks, chain_col_blocks(ks, in.ccol));
    const int64_t waves = std::max<int64_t>(1, std::min(per, (int64_t)in.n_cu / kXcds * 4 * per_simd));
    std::vector<int32_t> passes((size_t)(kXcds * waves), 0);
    int64_t slots = 0, longest = 0;
    for (int64_t b = 0; b < nb; ++b) {
        int32_t &w = passes[(size_t)(b / per * waves + b % per % waves)];
        slots += c.blocks[(size_t)b].slots;
        longest = std::max<int64_t>(longest, w += (c.blocks[(size_t)b].slots + em - 1) / em);
    }
    const int64_t even = (per + waves - 1) / waves * ((slots + nb * em - 1) / (nb * em));
    return 0.8 * (double)std::max<int64_t>(0, longest - even) +
           std::max(0.0, (double)nb - (double)in.n / (double)per_block) / (4.0 * in.n_cu) * block_mfma_us(in, ks);
}

void build_chain_pack(const InspectorInput &in, Schedule &s, bool entries) {
    s.chain = ChainPack();
    const int64_t n = in.n;
    const int es = elem_size(in.dtype);
    if (in.b_is_sparse || n == 0 || in.nnz == 0) return;
    // only where the caller has left the whole choice to the library
    if (!s.automatic || in.col_slice || in.gather_slices || !in.whole_fast_mem) return;
    const int ks = chain_ksteps(in.dtype, in.bcol);
    if (ks == 0 || chain_lds_bytes(in.dtype, in.bcol, in.ccol) > in.fast_mem_bytes) return;
    // (the kernel stores D through 32-bit byte offsets, in whole 16-byte pieces)
    if (in.ccol < vec_elems(in.dtype) || n * in.ccol * es >= ((int64_t)1 << 32) - 64) return;
    if (s.far_rows || one_pass_us(in, (double)in.nnz) >= two_wavefronts_us(in)) return;
    auto len = [&](int64_t j) { return (int64_t)in.rowptr[j + 1] - in.rowptr[j]; };
    int64_t longest = 0;
    for (int64_t j = 0; j < n; ++j) longest = std::max(longest, len(j));
    if (longest > kChainLongRow) return;
    // few blocks: rows are cut into parts so that there are about two waves per compute unit
    int slog = 0;
    while (slog < kChainMaxCut && ((n << slog) + 15) / 16 < 2 * (int64_t)in.n_cu && (in.nnz / n >> slog) >= 6) ++slog;
    const int64_t per_block = 16 >> slog;
    // A block far longer than the others holds one wave up while the rest of the machine is done: its
    // rows are cut further, until it has at most twice as many slots as a pass or a row of mean length.
    ChainPack &c = s.chain;
    c.early = chain_early(in.dtype, ks, n, in.nnz, in.bcol, in.ccol);
    const int em = chain_entries(in.dtype, ks, c.early);
    const int64_t most_slots = 2 * std::max<int64_t>(em, in.nnz / n >> slog);
    // rows in their own order while that pads little, else sorted by length inside windows
    int64_t padded = 0;
    for (int64_t j0 = 0; j0 < n; j0 += per_block) {
        int64_t mx = 0;
        for (int64_t j = j0; j < std::min(n, j0 + per_block); ++j) mx = std::max(mx, len(j));
        padded += mx * per_block;
    }
    c.rows.resize((size_t)n);
    std::iota(c.rows.begin(), c.rows.end(), 0);
    if (padded > in.nnz + in.nnz / 4) {
        const int64_t window = 2048;
        for (int64_t j0 = 0; j0 < n; j0 += window)
            std::stable_sort(c.rows.begin() + j0, c.rows.begin() + std::min(n, j0 + window),
                             [&](int32_t x, int32_t y) { return len(x) > len(y); });
    }
    c.blocks.reserve((size_t)(n / per_block) + 16);
    int64_t slot = 0;
    for (int64_t q0 = 0; q0 < n;) {
        ChainBlock cb{};
        int64_t q1;
        int cut = slog;
        for (;; ++cut) {
            // (empty rows share no block with others: nothing of B may be read for them)
            int64_t mx = len(c.rows[(size_t)q0]);
            q1 = q0 + 1;
            while (q1 < n && q1 < q0 + (16 >> cut) && (len(c.rows[(size_t)q1]) == 0) == (mx == 0))
                mx = std::max(mx, len(c.rows[(size_t)q1++]));
            cb.slots = (int32_t)((mx + (1 << cut) - 1) >> cut);
            if (cb.slots <= most_slots || cut == kChainMaxCut) break;
        }
        cb.slot_base = (uint32_t)slot;
        cb.row_begin = (int32_t)q0;
        const int passes = (cb.slots + em - 1) / em;
        cb.info = cut | (passes ? (cb.slots + passes - 1) / passes : 0) << 3 | (int32_t)((q1 - q0) << 7);
        c.blocks.push_back(cb);
        slot += cb.slots;
        q0 = q1;
    }
    const int64_t nb = (int64_t)c.blocks.size();
    const double two = s.streaming ? streaming_wavefronts_us(in, ks) : two_wavefronts_us(in);
    // Columns scattered around the diagonal (no tile fuses anything: the plan streams) find their row of B
    // in the L2 while it lies within 1 MiB of the row's own; farther ones come at 11.5 TB/s.  Stencils find
    // theirs at any distance: their columns move along with the rows.  (us, one pass / two wavefronts:
    // 141435 rows of 6 columns up to 27624 rows away, fp32 128 -> 32, 56 / 41; 281094 rows of 16, up to
    // 15680 away, fp64 103 -> 48, 475 / 249; 400000 rows of 8, fp32 128 -> 64, up to 2000 away 128 / 149, 25000
    // 212 / 187.  Of 696 such matrices this moved 17 that were up to 1.9 times faster in two wavefronts, and
    // none that was not.)
    const double far = s.streaming ? s.far_b_share : 0.0;
    // (the few per cent by which the ends of a stencil's rows pad are in the fits)
    const double with_padding = 16.0 * (double)slot > 1.125 * (double)in.nnz ? 16.0 * (double)slot : (double)in.nnz;
    if (one_pass_us(in, with_padding, far) + one_pass_tail_us(in, c, ks, per_block) >= two) {
        c = ChainPack();
        return;
    }
    if (!entries) return;
    const int64_t end = slot + kChainSpareSlots;
    c.idx.resize((size_t)end * 16);
    c.vals.resize((size_t)end * 16 * es + kChainZeroRows * kChainRowBytes);
    std::memset(c.idx.data() + slot * 16, 0, (size_t)kChainSpareSlots * 16 * 4);
    std::memset(c.vals.data() + (size_t)slot * 16 * es, 0, (size_t)kChainSpareSlots * 16 * es + kChainZeroRows * kChainRowBytes);
    auto fill = [&](auto tag) {
        typedef decltype(tag) T;
        const T *vals = static_cast<const T *>(in.vals);
        T *out = reinterpret_cast<T *>(c.vals.data());
        for_each_item(nb, host_threads(in.nnz, nb, 64), [&](int64_t b) {
            const ChainBlock &cb = c.blocks[(size_t)b];
            const int sl_log = cb.info & 7, parts = 1 << sl_log, n_rows = cb.info >> 7;
            for (int v = 0; v < 16; ++v) {
                // (virtual rows past the block's end repeat its last row; they are not stored)
                const int ri = std::min(v >> sl_log, n_rows - 1);
                const int64_t j = c.rows[(size_t)(cb.row_begin + ri)], k0 = in.rowptr[j], ln = len(j);
                const int64_t p0 = (int64_t)(v & (parts - 1)) * cb.slots;
                for (int64_t sl = 0; sl < cb.slots; ++sl) {
                    const int64_t at = ((int64_t)cb.slot_base + sl) * 16 + v, k = p0 + sl;
                    c.idx[(size_t)at] = k < ln ? in.colidx[k0 + k] : kChainPad;
                    out[at] = k < ln ? vals[k0 + k] : T(0);
                }
            }
        });
    };
    if (in.dtype == TF_F64) fill(double());
    else fill(float());
}

// A graph whose D1 rows are wider than the rows of B: the second wavefront gathers rows of cCol columns
// where the other order of the two products, Y = A B and then D = Y C, gathers rows of bCol.  All else
// is the same traffic (one n x bCol array read, one intermediate array written, D written), so the
// narrower gather decides; rows that do not end on whole half cache lines touch about another half line.
// Drawn at a fifth narrower; measured beyond (graphs, us per execution before -> after): fp32 131072
// rows 64 -> 128 160 -> 104, 382143 rows 32 -> 92 385 -> 157, fp64 142709 rows 64 -> 128 231 -> 220.
// Y takes the place of D1 in the plan's workspace.
void choose_gather_first(const InspectorInput &in, Schedule &s) {
    const int64_t n = in.n, es = elem_size(in.dtype);
    if (in.b_is_sparse || n == 0 || in.nnz == 0) return;
    // only where the caller has left the whole choice to the library
    if (!s.automatic || in.col_slice || in.gather_slices || !in.whole_fast_mem) return;
    if (!s.chain.blocks.empty() || !s.streaming) return;
    if (n > (int64_t)kInfoSlotMask || n * in.bcol > s.d1.rows * in.ccol) return;
    auto touched = [&](int64_t cols) { return cols * es % 64 ? cols * es + 64 : cols * es; };
    s.gather_first = 5 * touched(in.bcol) <= 4 * touched(in.ccol);
}

void build_gather_first(const InspectorInput &in, Schedule &s, bool have_all) {
    const int64_t n = in.n, es = elem_size(in.dtype);
    const D1Layout b = gather_first_slices(in.dtype, n, in.bcol, s.reuse);
    const PackRules rules = pack_rules(in, in.bcol, in.nnz, b), all_rules = pack_rules(in, in.ccol, in.nnz, s.d1);
    // (the sums and counts of cut rows of `all` have the places that rows of D1 need)
    s.gather_first_shares = have_all && rules.nr == all_rules.nr && rules.counts <= all_rules.counts &&
                            b.columns() <= s.d1.columns();
    if (!s.gather_first_shares) {
        std::vector<int32_t> all((size_t)n);
        std::iota(all.begin(), all.end(), 0);
        pack_rows(in.rowptr, in.colidx, static_cast<const unsigned char *>(in.vals), (int)es, std::move(all),
                  rules, [](int32_t c) { return c; }, s.gf);
    }
    s.gf_info.resize((size_t)n);
    for (int64_t j = 0; j < n; ++j)
        s.gf_info[(size_t)j] = in.rowptr[j + 1] > in.rowptr[j] ? kInfoSpill | (uint32_t)j : kInfoZero;
}

// us of a chain with CSR B over tiles, and as the two operations over all rows, D1 = B C and D = A D1; rows of B taken
// to be as long as those of A.  A compute unit works on a tile at a time, through a chain of barriers and dependent
// loads: a last round of a few tiles takes as long as a full one.  The pair gathers without barriers, and writes and
// reads all of D1.  Coefficients: fit to 170 bands and stencils of 2 to 49 entries a row, 6 to 140 columns, both types, 3
// to 80 MB of D1.  On 184 others the way it chooses takes 1.1 % more than the better one on average, 37 % at the worst; a
// limit on D1 that grows with the entries per row and the rows written again 2.2 and 52 %, one of 12 MB 13 and 94 %.
// (us, tiles / pair: band of 11 entries a row, fp64, 159683 x 37, 47 MB, 128 / 95; of 7, 27863 x 64, 14 MB, 18.1 / 19.2; of
// 9, fp32, 298330 x 29, 35 MB, 59 / 39; of 3, fp64, 91127 x 34, 25 MB, 24 / 34; 3D stencil, fp32, 32^3 x 80 31 / 19, 66^3 x 64,
// 74 MB, 70 / 86; 2D stencil, fp64, 246^2 x 32 24.6 / 18.7, 419^2 x 32 38 / 41.)
static double csr_tiles_us(const InspectorInput &in, const Schedule &s) {
    const double gathered = 1e-6 * (double)in.nnz * (double)in.ccol * elem_size(in.dtype);
    const double tiles = (double)std::max<int64_t>(1, (int64_t)s.tile_first_ptr.size() - 1);
    const double rounds = std::ceil(tiles * s.n_slices / std::max(1, in.n_cu));
    return 9.6 + 0.054 * gathered + rounds * (16.7 * gathered / (tiles * s.n_slices) + 0.77e-3 * (double)in.nnz / tiles);
}
static double csr_pair_us(const InspectorInput &in, const Schedule &s) {
    const double es = elem_size(in.dtype);
    return 6.3 + 0.082e-6 * (double)in.nnz * (double)in.ccol * es + 0.49e-6 * (double)(in.n * s.d1.columns()) * es;
}
bool plain_pair_is_faster(const InspectorInput &in, const Schedule &s) {
    if (!in.b_is_sparse || in.n == 0 || in.nnz == 0 || s.streaming) return false;
    // only where the caller has left the whole choice to the library
    if (!s.automatic || in.col_slice || in.gather_slices || !in.whole_fast_mem || (in.flags & TF_FLAG_SKIP_UNREAD))
        return false;
    // (what a plan keeps in device memory for it: rows as the workspace lays them out, padded where they reach far)
    if (in.n * s.d1.columns() * elem_size(in.dtype) > 80000000) return false;
    // (the tiles where there is little between them: they need no array of all rows)
    return csr_pair_us(in, s) < 0.94 * csr_tiles_us(in, s);
}

void build_baseline_pack(const InspectorInput &in, Schedule &s) {
    std::vector<int32_t> all((size_t)in.n);
    std::iota(all.begin(), all.end(), 0);
    pack_rows(in.rowptr, in.colidx, static_cast<const unsigned char *>(in.vals), elem_size(in.dtype), std::move(all),
              pack_rules(in, in.ccol, in.nnz, s.d1), [](int32_t c) { return c; }, s.all);
}

}  // namespace tf
