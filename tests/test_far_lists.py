"""CPU tests of the numbers behind the lists of k_far_gather (csrc/far_lists.h, used by the kernels and the host):
where the chunks of the buffer begin, for far entries anywhere among the rows and up to the largest matrix; and the
steps of the lists' conversion and of the gathering, one after the other as the kernels take them, every access
checked, with an incomplete last workgroup, x around the edges of its blocks, blocks and pieces without entries, and
several chunks."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHUNKS = r"""
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "far_lists.h"
// far(g): the far entries of workgroup g.  Every chunk has segments, all are covered, and with its padding it fits the buffer.
template <typename F>
static int check(const char* what, int groups, int value_bytes, F far) {
    std::vector<uint32_t> base;
    uint32_t total = 0;
    for (int g = 0; g < groups; g++) { base.push_back(total); total += uint32_t(far(g)); }
    base.push_back(total);
    const int segments = (groups + FAR_SEGMENT - 1) / FAR_SEGMENT, chunks = far_chunks(total, value_bytes);
    const auto segment_base = [&](int s) { return s < segments ? base.at(size_t(s) * FAR_SEGMENT) : total; };
    bool ok = chunks >= 1 && chunks <= FAR_MAX_CHUNKS && far_chunk_segment(base.data(), segments, total, chunks, 0) == 0;
    for (int c = 0, first = 0; ok && c < chunks; c++) {
        const int last = far_chunk_segment(base.data(), segments, total, chunks, c + 1);
        const int64_t most = int64_t(segment_base(last)) - segment_base(first) + FAR_MAX_BLOCKS * (FAR_PAD - 1);
        ok = last > first && most * value_bytes <= FAR_BUFFER_BYTES && (c + 1 < chunks || last == segments);
        if (!ok) std::printf("%s: %d groups, %u entries of %d bytes, chunk %d of %d: segments %d to %d of %d, %lld entries\n", what, groups, total, value_bytes, c, chunks, first, last, segments, (long long)most);
        first = last;
    }
    return ok ? 0 : 1;
}
int main() {
    const int most = 0x7fffffff / FAR_ENTRIES;
    int bad = 0;
    for (int value_bytes : {4, 8})
        for (int groups : {1, 63, 64, 65, 1000, 16604, 16640, 65537, most}) {
            bad |= check("all", groups, value_bytes, [](int) { return FAR_ENTRIES; });
            bad |= check("none", groups, value_bytes, [](int) { return 0; });
            bad |= check("first half", groups, value_bytes, [=](int g) { return g < groups / 2 ? FAR_ENTRIES : 0; });
            bad |= check("last tenth", groups, value_bytes, [=](int g) { return g >= groups - groups / 10 ? FAR_ENTRIES : 0; });
            bad |= check("middle", groups, value_bytes, [=](int g) { return g > groups / 3 && g < groups / 2 ? FAR_ENTRIES : g % 3; });
            bad |= check("every tenth segment", groups, value_bytes, [](int g) { return g / FAR_SEGMENT % 10 == 9 ? FAR_ENTRIES : 0; });
            bad |= check("uneven", groups, value_bytes, [](int g) { return int(uint32_t(g) * 2654435761u >> 19); });
        }
    return bad;
}
"""

LISTS = r"""
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "far_lists.h"
static uint32_t seed = 1;
static uint32_t draw() { return seed = seed * 1664525u + 1013904223u, seed >> 8; }
static uint32_t padded(uint32_t v) { return (v + FAR_PAD - 1) / FAR_PAD * FAR_PAD; }
// entries: of the whole tiles.  column(k): the column of entry k, -1 where it is near.
template <typename F>
static int check(const char* what, size_t entries, int n, int shift, int chunks, int pieces, F column) {
    const int cols_per_block = 1 << shift, blocks = (n + cols_per_block - 1) / cols_per_block;
    const int groups = int((entries + FAR_ENTRIES - 1) / FAR_ENTRIES), segments = (groups + FAR_SEGMENT - 1) / FAR_SEGMENT;
    std::vector<int32_t> col(entries);
    for (size_t k = 0; k < entries; k++) col[k] = column(k);
    // k_far_count
    std::vector<uint16_t> counts(size_t(groups) * blocks);
    std::vector<uint32_t> base(groups + 1);
    for (int g = 0; g < groups; g++)
        for (size_t k = size_t(g) * FAR_ENTRIES; k < entries && k < size_t(g + 1) * FAR_ENTRIES; k++)
            if (col[k] >= 0) counts.at(size_t(g) * blocks + (col[k] >> shift))++, base.at(g)++;
    // k_far_segments
    std::vector<uint32_t> sums(size_t(segments) * blocks);
    for (int g = 0; g < groups; g++)
        for (int b = 0; b < blocks; b++) sums.at(size_t(g / FAR_SEGMENT) * blocks + b) += counts.at(size_t(g) * blocks + b);
    uint32_t total = 0;
    for (int g = 0; g < groups; g++) { const uint32_t v = base[g]; base[g] = total; total += v; }
    base[groups] = total;
    // k_far_bases
    std::vector<uint32_t> range(size_t(chunks) * (blocks + 1)), list(chunks);
    std::vector<int> end(chunks);
    for (int c = 0; c < chunks; c++) {
        const int s0 = far_chunk_segment(base.data(), segments, total, chunks, c), s1 = far_chunk_segment(base.data(), segments, total, chunks, c + 1);
        uint32_t at = 0;
        for (int b = 0; b < blocks; b++) {
            uint32_t all = 0;
            for (int s = s0; s < s1; s++) all += sums.at(size_t(s) * blocks + b);
            range.at(size_t(c) * (blocks + 1) + b) = at;
            uint32_t to = at;
            for (int s = s0; s < s1; s++) { const uint32_t v = sums.at(size_t(s) * blocks + b); sums.at(size_t(s) * blocks + b) = to; to += v; }
            at += padded(all);
        }
        range.at(size_t(c) * (blocks + 1) + blocks) = list[c] = at;
        end[c] = s1;
    }
    // k_far_starts
    std::vector<uint32_t> starts(size_t(groups) * blocks);
    for (int s = 0; s < segments; s++)
        for (int b = 0; b < blocks; b++) {
            uint32_t at = sums.at(size_t(s) * blocks + b);
            for (int g = s * FAR_SEGMENT; g < groups && g < (s + 1) * FAR_SEGMENT; g++) { starts.at(size_t(g) * blocks + b) = at; at += counts.at(size_t(g) * blocks + b); }
        }
    // k_far_place
    size_t all_cols = 0, most = 0;
    std::vector<size_t> first(1);
    for (int c = 0; c < chunks; c++) { first.push_back(all_cols += list[c]); if (list[c] > most) most = list[c]; }
    std::vector<uint32_t> src(total);
    std::vector<uint16_t> place(total), cols(all_cols, 0xffff);
    for (int g = 0; g < groups; g++) {
        size_t my_first = 0;
        for (int c = 0; end.at(c) <= g / FAR_SEGMENT; c++) my_first += list.at(c);
        std::vector<uint32_t> next(blocks), from(blocks);
        uint32_t before = 0;
        for (int b = 0; b < blocks; b++) {
            next[b] = before;
            from[b] = starts.at(size_t(g) * blocks + b) - before;
            before += counts.at(size_t(g) * blocks + b);
        }
        for (size_t k = size_t(g) * FAR_ENTRIES; k < entries && k < size_t(g + 1) * FAR_ENTRIES; k++) {
            if (col[k] < 0) continue;
            const uint32_t q = next.at(col[k] >> shift)++, to = from.at(col[k] >> shift) + q;
            src.at(base[g] + q) = to;
            place.at(base[g] + q) = uint16_t(k % FAR_ENTRIES);
            cols.at(my_first + to) = uint16_t(col[k] & (cols_per_block - 1));
        }
    }
    // k_far_gather and the product, chunk after chunk through one buffer: x of a column is its number
    std::vector<int64_t> buffer(most, -1);
    for (int c = 0; c < chunks; c++) {
        std::vector<int> written(list[c]);
        for (int b = 0; b < blocks; b++)
            for (int piece = 0; piece < pieces; piece++) {
                const FarPiece mine(range.at(size_t(c) * (blocks + 1) + b), range.at(size_t(c) * (blocks + 1) + b + 1), piece, pieces);
                if (mine.empty()) continue;
                if (mine.begin % 2 || mine.end % 2 || first[c] % 8) return std::printf("%s: a pair across a piece's edge\n", what), 1;
                for (uint32_t k = mine.begin; k < mine.end; k++) buffer.at(k) = int64_t(b) * cols_per_block + cols.at(first[c] + k), written.at(k)++;
            }
        for (uint32_t k = 0; k < list[c]; k++)
            if (written[k] != 1) return std::printf("%s: value %u of chunk %d written %d times\n", what, k, c, written[k]), 1;
        for (int g = (c ? end[c - 1] : 0) * FAR_SEGMENT; g < groups && g < end[c] * FAR_SEGMENT; g++) {
            std::vector<int64_t> got(FAR_ENTRIES, -1);
            for (uint32_t k = base[g]; k < base[g + 1]; k++) got.at(place.at(k)) = buffer.at(src.at(k));
            for (size_t k = size_t(g) * FAR_ENTRIES; k < entries && k < size_t(g + 1) * FAR_ENTRIES; k++)
                if (got.at(k % FAR_ENTRIES) != col[k]) return std::printf("%s: entry %zu got %lld, not %d\n", what, k, (long long)got[k % FAR_ENTRIES], col[k]), 1;
        }
    }
    return 0;
}
int main() {
    int bad = 0;
    for (int shift : {14, 15})
        for (int n : {1, (1 << shift) - 1, 1 << shift, (1 << shift) + 1, (7 << shift) + 5, 40 << shift}) {
            const auto anywhere = [=](size_t) { return int32_t(draw() % uint32_t(n)); };
            bad |= check("anywhere", 700 * 512, n, shift, 1, 1, anywhere);
            bad |= check("pieces", 700 * 512 + 512, n, shift, 1, 6, anywhere);
            bad |= check("few", 3 * 512, n, shift, 1, 256, [=](size_t k) { return k % 7 ? -1 : int32_t(draw() % uint32_t(n)); });
            bad |= check("one block", 90 * 512, n, shift, 1, 3, [=](size_t k) { return k % 2 ? -1 : n - 1 - int32_t(k % uint32_t(n < 5 ? n : 5)); });
            bad |= check("none", 90 * 512, n, shift, 1, 3, [](size_t) { return -1; });
        }
    const int n = (9 << 14) + 77;
    const size_t entries = size_t(6) * FAR_SEGMENT * FAR_ENTRIES + 11 * 1024;
    for (int chunks : {2, 3}) {
        bad |= check("chunks", entries, n, 14, chunks, 2, [=](size_t) { return int32_t(draw() % uint32_t(n)); });
        bad |= check("chunks, first half", entries, n, 14, chunks, 2, [=](size_t k) { return k < entries / 2 ? int32_t(draw() % uint32_t(n)) : -1; });
        bad |= check("chunks, last half", entries, n, 14, chunks, 2, [=](size_t k) { return k >= entries / 2 ? int32_t(draw() % uint32_t(n)) : -1; });
    }
    return bad;
}
"""


@pytest.mark.parametrize("program", ["CHUNKS", "LISTS"])
def test_far_lists(tmp_path, program):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    src, exe = tmp_path / "far_lists.cpp", tmp_path / "far_lists"
    src.write_text(globals()[program])
    r = subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-D_GLIBCXX_ASSERTIONS", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "paper_1503_05032_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True, stdin=subprocess.DEVNULL, timeout=120)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, stdin=subprocess.DEVNULL, timeout=120)
    assert r.returncode == 0, (r.stdout, r.stderr)
