"""Index arithmetic that the kernels share with the host, at sizes whose arrays no test would allocate: small C++
programs over the library's internal header."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_00243_amd", "csrc")


def run_cpp(tmp_path, body):
    """Compiles and runs `body` as main(); CHECK(x) ends it with the line number."""
    src, exe = str(tmp_path / "main.cpp"), str(tmp_path / "main")
    with open(src, "w") as f:
        f.write('#include <cstdio>\n#include "tf_internal.h"\nusing namespace tf;\n'
                "#define CHECK(x) do { if (!(x)) { std::printf(\"line %d: %s\\n\", __LINE__, #x); return 1; } } while (0)\n"
                "int main() {\n" + body + "\nreturn 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, src,
                    "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr


def test_rows_beyond_the_slot_bits_of_an_info_word(tmp_path):
    """Without info words row j of B C goes to slot j, up to the last row that a plan takes, and nowhere else; with
    them to the slot in the word."""
    run_cpp(tmp_path, """
    const int64_t rows[] = {0, 1, ((int64_t)1 << 28) - 1, (int64_t)1 << 28, ((int64_t)1 << 29) + 5, ((int64_t)1 << 30) + 7,
                            ((int64_t)1 << 31) - 3};
    for (int64_t j : rows) {
        const uint32_t info = d1_info(false, 0);
        CHECK(info & kInfoSpill);
        CHECK(!(info & (kInfoDirect | kInfoZero | kInfoSkip)));
        CHECK(d1_slot(false, info, j) == j);
        const uint32_t given = kInfoDirect | kInfoSpill | 77u;
        CHECK(d1_info(true, given) == given && d1_slot(true, given, j) == 77);
    }""")


def test_rows_and_entries_at_the_end_of_32_bits(tmp_path):
    """Blocks cover the rows once, numbers past the end are none; a row that begins near the last possible entry has
    its own entries and no others, however long the rows beside it are.  (In 64 bits here, to compare with.)"""
    run_cpp(tmp_path, """
    for (uint32_t n : {1u, 63u, 64u, 1000u, 0x7fffffbfu, 0x7ffffffeu})
        for (uint32_t nr : {1u, 2u, 8u, 64u}) {
            const CsrBlocks b{n, nr};
            const uint64_t count = ((uint64_t)n + nr - 1) / nr, eighth = (count + 7) / 8;
            CHECK(b.count() == count && b.eighth() == eighth);
            for (uint64_t e = 1; e <= 8; ++e) CHECK(b.end(e) == (e * eighth < count ? e * eighth : count));
            for (uint64_t u : {(uint64_t)0, count / 2, count - 1, count})
                for (uint64_t v = 0; v < nr; ++v) {
                    CHECK(b.has(u, v) == (u * nr + v < n));
                    CHECK(b.row(u, v) == (u * nr + v < n ? u * nr + v : n - 1));
                }
        }
    for (int64_t begin : {(int64_t)0, (int64_t)5, (int64_t)0x7ffffff0, (int64_t)0x7ffffffe})
        for (int64_t len : {0, 1, 7, 15})
            for (int64_t s : {(int64_t)0, (int64_t)1, (int64_t)8, (int64_t)16, (int64_t)1 << 20, (int64_t)0x7fffffff,
                              (int64_t)0x7fffffff + 7}) {
                const int64_t end = begin + len <= 0x7fffffff ? begin + len : 0x7fffffff;
                CHECK(has_entry((int32_t)begin, (int32_t)end, (uint32_t)s) == (begin + s < end));
            }""")


def test_every_block_is_taken_once_and_long_rows_by_different_waves(tmp_path):
    """CsrWalk over ranges of all lengths; rows whose entries fall with the bits set in their number (the expected
    degrees of a recursive graph, largest at multiples of the powers of two): the busiest wave has about twice the
    longest row or its share at most; at a fixed place in every round it has 4 to 7 times that."""
    run_cpp(tmp_path, """
    for (uint32_t waves : {4u, 8u, 12u, 256u, 320u, 512u})
        for (uint32_t count : {1u, 3u, 4u, 5u, 511u, 512u, 513u, 4096u, 131072u}) {
            std::vector<int> taken(count, 0);
            int64_t busiest = 0, all = 0, longest = 0;
            for (uint32_t w = 0; w < waves; ++w) {
                int64_t passes = 0;
                uint32_t last = 0;
                for (CsrWalk u{w, w}; u.at < count; u = u.next(waves)) {
                    CHECK(u.place < waves && (u.at == w || u.at > last));
                    last = u.at;
                    ++taken[u.at];
                    double entries = 32.0 * count;
                    for (uint32_t k = u.at; k; k &= k - 1) entries *= 0.32;
                    const int64_t mine = 1 + (int64_t)entries / 8;
                    passes += mine;
                    longest = mine > longest ? mine : longest;
                }
                busiest = passes > busiest ? passes : busiest;
                all += passes;
            }
            for (int k : taken) CHECK(k == 1);
            // (launches of several blocks a wave have 128 waves and more on an XCD)
            if (waves >= 128) CHECK(busiest <= 2.25 * (longest > all / waves ? longest : all / waves));
        }""")
