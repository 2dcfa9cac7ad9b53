"""How the sort cuts a long list into runs and merge groups (sort_cut), compiled for the host: the
runs cover the list, none is longer than asked, and all runs and all groups of a pass have the same
length but for the odd keys (a short one would hold one workgroup up)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if shutil.which("g++") is None:
    pytest.skip("no host C++ compiler", allow_module_level=True)

PROGRAM = r"""
#include "fc_common.h"
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#define CHECK(x) do { if (!(x)) { printf("m %d most %d launched %d blocks %d: %s\n", m, most, launched, blocks, #x); return 1; } } while (0)
static int check(int m, int most, int launched, int blocks) {
    const fc::SortCut c = fc::sort_cut(m, most, launched, blocks);
    if (m <= 0) { CHECK(c.runs == 0 && c.passes == 0); return 0; }
    // more runs than the passes take: each workgroup merges its own share first
    const int least = (m + most - 1) / most;
    const bool shares = launched > 0 && least > (launched < 3 ? 256 : 512);
    CHECK(c.runs >= (shares ? blocks : least) && c.passes >= 0 && c.passes <= launched);
    CHECK((c.passes == 0) == (c.runs == 1 || launched == 0) && (shares || (c.runs == 1) == (m <= most)));
    CHECK(c.start(0) == 0 && c.start(c.runs) == m && c.len >= 1 && (shares || c.len + (c.rem > 0) <= most));
    CHECK(c.rem < c.runs && c.start(c.runs) - c.start(c.runs - 1) >= c.start(1) - 1);
    int u = 1;
    for (int p = 0; p + 1 < c.passes; ++p) {
        const int fan = p == 0 ? c.fan : c.fan2;
        CHECK(fan >= 2 && c.runs % (u * fan) == 0);          // whole groups
        u *= fan;
        // the last group is as long as the first, but for a key a run
        CHECK(c.start(c.runs) - c.start(c.runs - u) >= c.start(u) - u);
    }
    // groups of nearly the least size for these passes, and few more runs than asked
    if (c.passes >= 2 && !shares) CHECK(c.runs / u <= c.fan + 1 && c.runs <= least + least / 6 + 1);
    if (c.passes == 1) CHECK(c.runs <= (blocks > 256 ? blocks : 256));
    return 0;
}
int main() {
    const int mosts[] = {2048, 4096};
    for (int most : mosts)
        for (int launched = 0; launched <= 3; ++launched)
            for (int blocks : {1, 2, 15, 16, 170, 256, 512}) {
                for (int m = -1; m < 300000; m += m < 20000 ? 1 : 37) if (check(m, most, launched, blocks)) return 1;
                for (long long m = 300000; m < (1ll << 29); m += m / 97 + 1)
                    if (check((int)m, most, launched, blocks)) return 1;
                if (check(5218382, most, launched, blocks) || check((1 << 29) - 1, most, launched, blocks)) return 1;
            }
    puts("ok");
}
"""


def test_sort_cut(tmp_path):
    src, exe = tmp_path / "cut.cpp", tmp_path / "cut"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    "-I", os.path.join(ROOT, "paper_2606_04801_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
