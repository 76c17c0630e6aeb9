"""The index arithmetic of the device builder and of the cut's long rows
(csrc/slot_index.h) on the host, where entry and slot indices reach INT_MAX:
no device array of that size is needed to check it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HEAD = r"""
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "slot_index.h"
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)
"""

PROGRAMS = {
    # sorted keys 2 * i, seen only through an accessor that stays in lo..hi
    "search": r"""
struct Keys {
    int lo, hi;
    unsigned long long operator[](int i) const { CHECK(i >= lo && i < hi); return 2ull * (unsigned)i; }
};
int main() {
    const int ends[] = {0, 1, 7, 1 << 30, (1 << 30) + 5, INT_MAX - 1, INT_MAX};
    for (int lo : ends)
        for (int hi : ends) {
            if (hi < lo) continue;
            const Keys k{lo, hi};
            for (int i : {lo, lo + (hi - lo) / 2, hi - 1}) {
                if (i < lo || i >= hi) continue;
                CHECK(mf::first_at_least(k, lo, hi, 2ull * i) == i);
                CHECK(mf::first_at_least(k, lo, hi, 2ull * i + 1) == i + 1);
            }
            CHECK(mf::first_at_least(k, lo, hi, ~0ull) == hi);
            CHECK(mf::first_at_least(k, lo, hi, 0ull) == lo);
        }
}
""",
    # rows that end at INT_MAX, by 8 lanes (free slots) and by a workgroup
    "strided": r"""
int main() {
    for (int end : {INT_MAX, INT_MAX - 1, INT_MAX - 7, INT_MAX - 1024, 1000})
        for (int len : {0, 1, 7, 8, 9, 700})
            for (int step : {8, 1024}) {
                long long seen = 0, sum = 0;
                for (int lane = 0; lane < step; ++lane)
                    mf::strided((int64_t)end - len + lane, end, step, [&](int j) {
                        CHECK(j >= end - len && j < end && seen < 2000);
                        ++seen;
                        sum += j - (end - len);
                    });
                CHECK(seen == len && sum == (long long)len * (len - 1) / 2);
            }
}
""",
    # a workgroup's loads past the end of such a row read its last slot
    "last": r"""
int main() {
    for (int end : {INT_MAX, INT_MAX - 1, 5})
        for (int j0 : {end - 4, end - 1})
            for (int off : {0, 1, 3, 256, 768, 1024}) {
                const int j = mf::slot_or_last((int64_t)j0 + off, end);
                CHECK(j >= j0 && j < end && (j == end - 1 || j == j0 + off));
            }
}
""",
    # 8 threads for each of up to INT_MAX vertices
    "blocks": r"""
int main() {
    for (int64_t n : {0ll, 1ll, 32ll, 33ll, 1ll << 20, (1ll << 29) - 1, 1ll << 29, (long long)INT_MAX}) {
        const unsigned b = mf::stride_blocks(8 * n, 256);
        CHECK(b >= 1 && (unsigned long long)b * 256 < 1ull << 32);
        if (8 * n <= 1ll << 31) CHECK((int64_t)b * 256 >= 8 * n);
    }
}
""",
}


@pytest.mark.parametrize("name", PROGRAMS)
def test_index_limits(tmp_path, name):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(HEAD + PROGRAMS[name])
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-ftrapv",
                           "-I", os.path.join(ROOT, "paper_2511_01235_amd", "csrc"), "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
