"""The rules by which a launch is chosen: the header is plain arithmetic, so a host compiler runs it."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_01278_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "host_rules.hpp"
int main(int, char** v) {
  if (v[1][0] == 'm') printf("%d\n", pillar::merger_groups(atoll(v[2]), atoi(v[3]), atoi(v[4]), atoi(v[5]), 256));
  if (v[1][0] == 'b') printf("%d\n", pillar::draft_bypasses(atoll(v[2]), atoi(v[3]) != 0));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "rules")
    subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, str(d / "main.cpp"), "-o", exe], check=True)
    return lambda *args: int(subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True).stdout)


@pytest.fixture(scope="module")
def mergers(rule):
    return lambda *args: rule("m", *args)


def test_mergers_only_where_they_take_two_turns_at_most(mergers):
    """256 compute units.  A turn of a pair's mergers is four rows per merger and 512 threads; with more than two turns of 1024 threads, 96
    pairs with 64 rows took 39 us where they take 36 without mergers."""
    for pairs in (1, 8, 40, 64, 80, 85, 86, 88, 96, 97, 102, 103, 128, 129, 200):
        for rows in (1, 4, 5, 16, 20, 32, 33, 36, 40, 48, 64):
            for threads in (512, 1024):
                n = mergers(pairs, 4096, rows, threads)
                assert 0 <= n <= -(-rows // (threads // 128))
                assert (n > 0) == (pairs <= 128 and rows <= 16 * (2 * (256 - pairs) // pairs)), (pairs, rows, threads, n)
    assert mergers(96, 4096, 64, 1024) == 0 and mergers(88, 4096, 64, 512) == 0 and mergers(85, 4096, 64, 1024) == 4
    assert mergers(96, 4096, 48, 1024) == 3 and mergers(102, 4096, 48, 1024) == 3 and mergers(103, 4096, 48, 1024) == 0
    # contexts of up to n chunks of 8192 tokens take n workgroups per pair
    assert mergers(8, 16 * 8192, 20, 1024) > 0 and mergers(8, 16 * 8192 + 1, 20, 1024) == 0


def test_draft_rows_bypass_beyond_96_mb(rule):
    bypass = lambda list_rows, fp8: bool(rule("b", list_rows, int(fp8)))
    line = (96 << 20) // 512
    assert not bypass(line, False) and bypass(line + 1, False) and not bypass(2 * line, True) and bypass(2 * line + 1, True)
    assert bypass(1 << 40, False) and not bypass(0, False)
