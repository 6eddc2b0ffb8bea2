"""The planners' stable sort, compiled by the host compiler from the header that they use."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_01381_amd", "csrc")


def _run(tmp_path, body):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "sort.cpp", tmp_path / "sort"
    src.write_text('#include <stdio.h>\n#include <random>\n#include "host_sort.hpp"\nusing namespace adaqp;\n'
                   '#define CHECK(x) do { if (!(x)) { printf("line %d: %s\\n", __LINE__, #x); return 1; } } while (0)\n'
                   "static long moves = 0;\n"
                   "struct Counted {\n"
                   "    int32_t at = 0;\n"
                   "    Counted() = default;\n"
                   "    Counted(const Counted &) = default;\n"
                   "    Counted &operator=(const Counted &from) { at = from.at; ++moves; return *this; }\n"
                   "};\n"
                   "int main() {\n" + body + "\nreturn 0; }\n")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wno-class-memaccess", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout


@pytest.mark.parametrize("n", [256, 257, 5000])
def test_digits_in_which_all_keys_agree_cost_no_pass(tmp_path, n):
    """Keys of 27 and more bits whose low ones are the same in all of them (floats that came from 16 bits) are moved once less than
    others, and keys that only differ in a few bits in the middle once."""
    _run(tmp_path, f"""
    std::mt19937 draw(7);
    const size_t n = {n};
    struct {{ uint32_t range, apart, lo; long passes; }} kinds[] = {{{{1u << 27, 1, 0, 3}}, {{1u << 11, 1u << 16, 0x1fff, 2}}, {{4, 1u << 20, 5, 1}},
                                                                  {{0xffffffffu, 1, 0, 3}}, {{1, 1, 77, 0}}}};
    for (auto kind : kinds) {{
        std::vector<KeyedIndex<Counted>> items(n), other(n), want;
        for (size_t i = 0; i < n; ++i) {{
            items[i].key = kind.lo + kind.apart * (i == 0 ? 0 : i == 1 ? kind.range - 1 : draw() % kind.range);
            items[i].index.at = (int32_t)i;
        }}
        want = items;
        std::stable_sort(want.begin(), want.end(), [](const KeyedIndex<Counted> &x, const KeyedIndex<Counted> &y) {{ return x.key < y.key; }});
        moves = 0;
        sort_by_key(items.data(), other.data(), n);
        CHECK(moves == kind.passes * (long)n);
        for (size_t i = 0; i < n; ++i) CHECK(items[i].key == want[i].key && items[i].index.at == want[i].index.at);
    }}
    """)


@pytest.mark.parametrize("runs", [0, 1, 2, 3, 7, 64, 1000])
def test_merging_runs_moves_an_item_once_per_doubling(tmp_path, runs):
    """Runs of any lengths, empty ones among them, equal items too; as many comparisons as doublings of the number of runs times items."""
    _run(tmp_path, f"""
    static long compared;
    struct Item {{
        double key;
        bool operator<(const Item &other) const {{ ++compared; return key < other.key; }}
    }};
    std::mt19937 draw(11);
    const size_t runs = {runs};
    std::vector<Item> items;
    std::vector<size_t> ends;
    for (size_t q = 0; q < runs; ++q) {{
        std::vector<double> run(draw() % 5 == 0 ? 0 : draw() % 40);
        for (double &x : run) x = (double)(draw() % 500);
        std::sort(run.begin(), run.end());
        for (double x : run) items.push_back({{x}});
        ends.push_back(items.size());
    }}
    std::vector<double> want;
    for (const Item &item : items) want.push_back(item.key);
    std::sort(want.begin(), want.end());
    compared = 0;
    merge_runs(items, ends);
    long doublings = 0;
    while (((size_t)1 << doublings) < runs) ++doublings;
    CHECK(compared <= doublings * (long)items.size());
    for (size_t k = 0; k < want.size(); ++k) CHECK(items[k].key == want[k]);
    """)
