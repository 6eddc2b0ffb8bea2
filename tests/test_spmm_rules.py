"""Arithmetic of the sliced aggregation, compiled by the host compiler from the header that the kernel uses."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_01381_amd", "csrc")


def _run(tmp_path, body):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <stdio.h>\n#include <initializer_list>\n#include "spmm_rules.hpp"\nusing namespace adaqp;\n'
                   '#define CHECK(x) do { if (!(x)) { printf("line %d: %s\\n", __LINE__, #x); return 1; } } while (0)\n'
                   "int main() {\n" + body + "\nreturn 0; }\n")
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout


def test_buffer_extent(tmp_path):
    """No extent holds the offset that stands for "nothing to fetch", whatever column is added to it; every row's columns
    lie inside."""
    _run(tmp_path, """
    const int64_t cols[] = {0, 1, 2, 5, 1000, 1 << 20};
    const int64_t pitches[] = {32, 64, 608, 2048, 2080, 1000};
    for (int64_t n : cols) for (int64_t ld : pitches) {
        if (n * ld * 4 >= (int64_t)kOutside) continue;
        for (int32_t begin = 0; begin < 2048; begin += 32) {
            const uint32_t e = buffer_extent(n, ld, begin);
            CHECK(e <= kOutside);
            CHECK(n > 0 || e == 0);
            if (n > 0 && begin + 32 <= ld) CHECK((int64_t)e >= ((n - 1) * ld + 32) * 4 && (int64_t)e <= n * ld * 4);
        }
    }
    """)


def test_what_the_sliced_kernel_takes(tmp_path):
    """Never a call whose arrays may be NULL (no entries, no columns), nor one whose offsets do not fit 32 bits."""
    _run(tmp_path, """
    CHECK(sliced_takes(5, 1, 1, 32, false, 0, 32));
    CHECK(!sliced_takes(5, 0, 0, 64, false, 0, 64) && !sliced_takes(5, 0, 0, 64, true, 4, 64));
    CHECK(!sliced_takes(5, 0, 5, 64, false, 0, 64) && !sliced_takes(5, 5, 0, 64, false, 0, 64));
    const int64_t floats = (int64_t)kOutside / 4;
    CHECK(sliced_takes(5, 9, floats / 32 - 1, 32, false, 0, 32) && !sliced_takes(5, 9, floats / 32 + 1, 32, false, 0, 32));
    CHECK(!sliced_takes(5, 9, (int64_t)1 << 33, 32, false, 0, 32) && !sliced_takes(5, 9, 2, (int64_t)1 << 62, false, 0, 32));
    for (int64_t n = 1; n < ((int64_t)1 << 32); n = n * 5 / 4 + 1)        // what the search adds to a number of rows stays in 32 bits
        if (sliced_takes(n, 9, 10, 32, false, 0, 32)) {
            const int64_t step = (n + kProbes - 1) / kProbes;
            CHECK(n + kProbes - 1 <= INT32_MAX && n + step - 1 <= INT32_MAX && n + 64 <= INT32_MAX);
        }
    CHECK(sliced_takes(2000000000, 9, 10, 32, false, 0, 32) && !sliced_takes(INT32_MAX - 1, 9, 10, 32, false, 0, 32));
    CHECK(sliced_takes(5, 9, 10, 32, true, 4096, 32) && !sliced_takes(5, 9, 10, 32, true, (int64_t)1 << 32, 32));
    """)


def test_buffer_loads_carry_no_scalar_offset():
    """The scalar offset of a raw buffer load is not part of what is compared with the buffer's extent: a load that relies
    on that comparison must not use it."""
    calls = 0
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".hpp")):
            continue
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        for found in re.finditer(r"__builtin_amdgcn_raw_buffer_load_\w+\(", text):
            args, depth, at = [""], 0, found.end()
            while depth >= 0:
                c = text[at]
                depth += (c in "([{") - (c in ")]}")
                if depth == 0 and c == ",":
                    args.append("")
                elif depth >= 0:
                    args[-1] += c
                at += 1
            calls += 1
            assert len(args) == 4 and args[2].strip() == "0", f"{name}: scalar offset {args[2].strip()}"
    assert calls > 0


def test_cuts_of_the_sliced_kernel(tmp_path):
    """A cut is always one that the kernel has; and where launches were measured slower than along the merge path (few entries,
    short rows with a narrower slice, packed rows one line at a time, rows that share lines and too many columns), that
    path or another cut is taken."""
    _run(tmp_path, """
    for (int64_t rows : {1, 40, 2000, 60000, 300000, 2000000000}) for (int64_t degree : {0, 1, 5, 18, 64, 300, 30000})
        for (int64_t cols : {1, 700, 10241, 40001, 100000, 200001, 3000000}) for (int32_t lines = 1; lines <= 64; ++lines)
            for (int whole = 0; whole < 2; ++whole) for (int skewed = 0; skewed < 2; ++skewed) {
                const SlicedCut c = sliced_cut(rows, rows * degree, cols, lines, whole != 0, skewed != 0);
                CHECK((c.lines == 0) == (c.packed_lines == 0) && (c.lines == 0 || (c.n_blocks >= 1 && c.n_blocks <= 1024)));
                CHECK(c.lines == 0 || c.lines == 1 || c.lines == 2 || c.lines == 4);
                CHECK(c.packed_lines == 0 || c.packed_lines == 2 || c.packed_lines == 4);
                CHECK(whole || c.lines == 0 || c.lines == 4);
            }
    CHECK(sliced_cut(2000, 20656, 2600, 4, true, false).lines == 0);
    CHECK(sliced_cut(10000, 80000, 15000, 4, true, true).lines == 0);
    CHECK(sliced_cut(40000, 160000, 60000, 13, true, false).lines == 0);
    CHECK(sliced_cut(150000, 600000, 225000, 17, true, false).lines == 0);
    CHECK(sliced_cut(46921, 841725, 65616, 17, true, false).packed_lines == 4);
    CHECK(sliced_cut(40000, 2800000, 60000, 5, false, false).lines == 0);
    CHECK(sliced_cut(2500, 45000, 3750, 1, false, false).lines == 0);
    """)


def test_every_slice_task_is_taken_once(tmp_path):
    """Every share of every slice by exactly one workgroup, whatever the last slice's width, and no XCD with much more weight
    than another."""
    _run(tmp_path, """
    for (int packed = 0; packed < 2; ++packed)
        for (int32_t vpl : {1, 2, 4}) for (int32_t lines = 1; lines <= 64; ++lines)
            for (int32_t n_blocks : {1, 2, 3, 7, 8, 31, 64, 127, 170, 512, 2048}) {
                const SliceTasks t(lines, vpl, n_blocks, packed != 0);
                const int64_t n_tasks = (int64_t)((lines + vpl - 1) / vpl) * n_blocks;
                CHECK(t.first_task(0) == 0 && t.first_task(kXcds) == n_tasks);
                int64_t next = 0;
                for (int32_t x = 0; x < kXcds; ++x) {
                    CHECK(t.first_task(x) == next);
                    next = t.first_task(x + 1);
                    CHECK(next >= t.first_task(x) && next - t.first_task(x) <= t.most_per_xcd());
                    int64_t weight = 0;
                    for (int64_t k = t.first_task(x); k < next; ++k) weight += k < t.full ? t.whole_weight : t.rest_weight;
                    CHECK(weight <= t.all / kXcds + 1 + t.whole_weight);
                }
            }
    """)


def test_launches_of_planned_pieces_have_room(tmp_path):
    """Fewer than 2^32 threads, however many pieces and lines there are; a whole number of slices, at least one."""
    _run(tmp_path, """
    for (int32_t waves : {4, 8}) for (int packed = 0; packed < 2; ++packed) for (int32_t vpl : {1, 2, 4}) {
        const int64_t most = kMostPieces / waves;
        for (int64_t n = 1; n <= most; n = n < most && n * 5 / 4 + 1 > most ? most : n * 5 / 4 + 1) {
            const int64_t lines = pieces_lines(n, waves, vpl);
            CHECK(lines >= vpl && lines % vpl == 0);
            for (int64_t l = 1; l <= lines && l < INT32_MAX; l = l < 64 || l >= lines - 64 ? l + 1 : (2 * l < lines - 64 ? 2 * l : lines - 64))
                CHECK(SliceTasks((int32_t)l, vpl, (int32_t)n, packed != 0).most_per_xcd() * kXcds * waves * 64 < ((int64_t)1 << 32));
        }
    }
    """)
