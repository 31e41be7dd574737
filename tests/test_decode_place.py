"""Which workgroup of the draft step takes which (request, KV head, span): the header is plain arithmetic, so a host compiler runs it."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_01278_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "decode_place.hpp"
int main(int, char** v) {
  const unsigned batch = atoi(v[2]), heads = atoi(v[3]), nspan = atoi(v[4]);
  for (unsigned i = 0; i < batch * heads * nspan; ++i) {
    const pillar::DecPlace p = pillar::decode_place(atoi(v[1]) != 0, i, batch, heads, nspan);
    printf("%d %d %d\n", p.slot_b, p.g, p.sp);
  }
}
"""


@pytest.fixture(scope="module")
def place(tmp_path_factory):
    d = tmp_path_factory.mktemp("place")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "place")
    subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, str(d / "main.cpp"), "-o", exe], check=True)

    def run(fp8, batch, heads, nspan):
        text = subprocess.run([exe, str(int(fp8)), str(batch), str(heads), str(nspan)], check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in text.splitlines()]
    return run


@pytest.mark.parametrize("fp8", [False, True])
def test_every_span_is_taken_once(place, fp8):
    for batch in (1, 7, 8, 9, 16, 23, 64):
        for heads in (1, 3, 8):
            for nspan in (1, 2, 3, 4, 8):
                want = [(b, g, sp) for b in range(batch) for g in range(heads) for sp in range(nspan)]
                assert sorted(place(fp8, batch, heads, nspan)) == want
                if not fp8:
                    assert place(fp8, batch, heads, nspan) == want


@pytest.mark.parametrize("batch,long", [(8, {3}), (64, set(range(3, 64, 8))), (128, set(range(0, 128, 8))), (16, {0, 8}), (64, set())])
def test_long_lists_do_not_load_one_xcd(place, batch, long):
    """Lists of four spans among lists of one (fp8): no XCD, of eight that take the workgroups in turn, has more than half again the mean.
    With every eighth request's four spans on one XCD it had almost three times the mean, and 128 requests took 73 us instead of 51."""
    load = [0] * 8
    for i, (b, g, sp) in enumerate(place(True, batch, 8, 4)):
        load[i % 8] += sp < (4 if b in long else 1)
    assert max(load) <= 1.5 * sum(load) / 8


def test_heads_of_a_span_share_an_xcd(place):
    for nspan in (1, 4):
        seen = {}
        for i, (b, g, sp) in enumerate(place(True, 24, 8, nspan)):
            seen.setdefault((b, sp), set()).add(i % 8)
        assert all(len(x) == 1 for x in seen.values())
