"""The attention kernel with four wavefronts (128 query rows) per workgroup, pinned, on the problems that its other
forms are checked on: row counts around the edges of a tile, a half tile and a workgroup, running maxima raised inside the
pipelined loop, block lists of every block size (256: two workgroups share a row block), gather and scatter."""
import pytest

from tests import test_gpu_parity as par

pytestmark = pytest.mark.gpu

tsa = par.tsa


@pytest.fixture
def pair(tsa):
    tsa.tsa_bench_set_attend_form(3)
    yield 3
    tsa.tsa_bench_set_attend_form(0)


@pytest.mark.parametrize("Lc", [1, 31, 33, 64, 127, 128, 129, 191, 257, 1000])
@pytest.mark.parametrize("d", [64, 128])
def test_rows(tsa, pair, Lc, d):
    par.test_attend_matches_oracle(tsa, pair, 1, 4, 2, Lc, d)


def test_sweep_and_growing_logits(tsa, pair):
    par.test_attend_random_sweep(tsa, pair)
    par.test_attend_logits_growing_along_the_keys(tsa, pair)
    par.test_attend_large_logits_and_scale(tsa, pair)


@pytest.mark.parametrize("Lc,window,Bs", [(1000, 256, 64), (1300, 128, 128), (1500, 512, 256), (3000, 1024, 256)])
def test_block_lists(tsa, pair, Lc, window, Bs):
    par.test_attend_block_list(tsa, pair, Lc, window, Bs)


@pytest.mark.parametrize("B,Hq,Hkv,L,d,k,group_mode,with_blocks", [
    (1, 4, 2, 1500, 128, 700, 0, False), (2, 6, 2, 1203, 128, 333, 1, False), (1, 4, 4, 900, 64, 900, 0, False),
    (3, 2, 1, 777, 64, 200, 0, True), (1, 4, 2, 4001, 64, 130, 0, False), (2, 4, 2, 520, 128, 1, 0, False)])
def test_gather_and_scatter(tsa, pair, B, Hq, Hkv, L, d, k, group_mode, with_blocks):
    par.test_fused_path_equals_the_separate_calls(tsa, pair, B, Hq, Hkv, L, d, k, group_mode, with_blocks)
