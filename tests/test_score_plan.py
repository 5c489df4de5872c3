"""How a scoring call is cut into workgroups (csrc/score_plan.h, host code, compiled here): chunks twice as long, for the sake of
one launch less, are served by workgroups of fewer heads, so that the chip has no fewer of them than it had."""
import itertools
import os
import shutil
import subprocess

import pytest

from paper_2602_03216_amd import build

MAIN = r"""
#include "score_plan.h"
#include <cstdio>
int main() {
  int KVH, g, L, d, q;
  while (scanf("%d %d %d %d %d", &KVH, &g, &L, &d, &q) == 5) {
    const tsa::ScorePlan p = tsa::plan_score(KVH, g, L, d, q);
    printf("%d %d %d\n", p.chunk, p.nchunks, p.heads);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no host compiler")
    at = tmp_path_factory.mktemp("plan")
    (at / "main.cpp").write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-I", build.CSRC, str(at / "main.cpp"), "-o", str(at / "plan")], check=True)

    def run(shapes):
        text = "\n".join(" ".join(map(str, s)) for s in shapes)
        out = subprocess.run([str(at / "plan")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def _single(KVH, g, L, q):
    """the cut into chunks of single length: (chunk, chunks of all KV heads, heads per workgroup that suit it)"""
    resident = 512 if q <= 64 else 256
    chunk = min(max((L * KVH // resident + 127) // 128 * 128, 256), 8192)
    n = -(-L // chunk) * KVH
    heads = 4 if g >= 4 else 2 if g >= 2 else 1
    while heads > 1 and n * -(-g // heads) <= 128:
        heads //= 2
    return chunk, n, heads


def test_no_call_loses_workgroups_to_longer_chunks(plan):
    shapes = [s for s in itertools.product((1, 2, 3, 4, 6, 8, 10, 16, 32), (1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 32),
                                           (600, 3001, 8192, 8193, 9000, 10007, 12345, 16000, 16384, 20000, 32768, 65536, 131072), (64, 128), (1, 32, 33, 64, 65, 128))]
    longer = 0
    for (KVH, g, L, d, q), (chunk, n, heads) in zip(shapes, plan(shapes)):
        single, n_before, heads_before = _single(KVH, g, L, q)
        assert chunk % 128 == 0 and chunk >= 256 and n == -(-L // chunk) and heads in (1, 2, 4) and (heads == 1 or heads <= g)
        if chunk == single:
            assert heads == heads_before
            continue
        assert chunk == 2 * single and g >= 4 and heads <= 2 and n <= 32
        longer += 1
        # workgroups, without the idle slots of a last round of heads
        assert n * KVH * g / heads >= min(n_before * g / heads_before, 256), (KVH, g, L, d, q)
    assert longer > 100


@pytest.mark.parametrize("shape,longer", [
    ((1, 4, 8193, 64, 33), False), ((1, 4, 8193, 128, 128), False), ((1, 6, 10000, 128, 64), False),   # single heads already
    ((1, 8, 9000, 128, 64), True), ((2, 5, 9000, 128, 100), True), ((8, 4, 10007, 128, 64), True),
    ((8, 4, 10007, 128, 32), True), ((4, 4, 10000, 128, 32), False), ((8, 8, 14000, 128, 32), False), ((8, 8, 14000, 128, 33), True),
    ((1, 16, 12000, 128, 64), True), ((1, 32, 9000, 128, 64), False),
    ((8, 4, 8192, 128, 64), False), ((8, 4, 16385, 128, 64), False), ((8, 4, 20000, 128, 64), True), ((8, 4, 32768, 128, 64), False),
    ((8, 4, 32768, 64, 64), True)])
def test_where_chunks_are_twice_as_long(plan, shape, longer):
    KVH, g, L, d, q = shape
    (chunk, _, _), = plan([shape])
    assert chunk == _single(KVH, g, L, q)[0] * (2 if longer else 1)
