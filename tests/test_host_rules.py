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
int main(int argc, char** v) {
  if (v[1][0] == 'm') printf("%d\n", pillar::merger_groups(atoll(v[2]), atoi(v[3]), atoi(v[4]), atoi(v[5]), 256));
  if (v[1][0] == 'p') {                       // shift, tiles of every pair: slot, first tile, tiles of every piece
    const int shift = atoi(v[2]);
    int u0 = 0;
    for (int pair = 0; pair < argc - 3; ++pair) {
      const int tiles = atoi(v[3 + pair]), n = pillar::pieces_of(tiles, shift);
      for (int i = 0; i < n; ++i) {
        const int at = pillar::piece_begin(tiles, n, tiles / n, i);
        printf("%d %d %d\n", pair + pillar::first_slot(u0, shift) + i, at, pillar::piece_begin(tiles, n, tiles / n, i + 1) - at);
      }
      u0 += tiles;
    }
  }
  if (v[1][0] == 'b') printf("%d\n", pillar::draft_bypasses(atoll(v[2]), atoi(v[3]) != 0));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "rules")
    subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, str(d / "main.cpp"), "-o", exe], check=True)

    def run(*args):
        text = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in text.splitlines()]
    return run


@pytest.fixture(scope="module")
def mergers(rule):
    return lambda *args: rule("m", *args)[0][0]


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
    assert mergers(102, 1290, 40, 1024) == 3 and mergers(104, 1290, 40, 1024) == 0 and mergers(84, 1290, 64, 512) == 4 and mergers(86, 1290, 64, 512) == 0
    # contexts of up to n chunks of 8192 tokens take n workgroups per pair
    assert mergers(8, 16 * 8192, 20, 1024) > 0 and mergers(8, 16 * 8192 + 1, 20, 1024) == 0


def test_draft_rows_bypass_beyond_96_mb(rule):
    bypass = lambda list_rows, fp8: bool(rule("b", list_rows, int(fp8))[0][0])
    line = (96 << 20) // 512
    assert not bypass(line, False) and bypass(line + 1, False) and not bypass(2 * line, True) and bypass(2 * line + 1, True)
    assert bypass(1 << 40, False) and not bypass(0, False)


@pytest.mark.parametrize("shift", [1, 2, 3, 4, 5])
def test_pieces_of_a_pair_are_alike_and_have_slots_of_their_own(rule, shift):
    """Every tile once, no piece longer than 2^shift tiles or two tiles apart from another of its pair (18 tiles in two were 16 and 2), as few
    as that takes; slots grow along the layout and stay below pairs + pieces."""
    most = 1 << shift
    tiles = [1, 2, most - 1, most, most + 1, 18, 0, 0, 2 * most - 1, 2 * most, 2 * most + 1, 1, 1, 1, 5 * most + 3] + [(7 * i) % (3 * most) for i in range(200)]
    rows = rule("p", shift, *tiles)
    slots = [r[0] for r in rows]
    assert slots == sorted(set(slots)) and slots[-1] < len(tiles) + len(rows)
    at = iter(rows)
    for n in tiles:
        pieces = [next(at) for _ in range(-(-n // most))]
        end = 0
        for _, first, count in pieces:
            assert first == end and 0 < count <= most
            end += count
        assert end == n and (not n or max(p[2] for p in pieces) - min(p[2] for p in pieces) <= 1)
