"""The attention kernel with four wavefronts (128 query rows) per workgroup, pinned, at the edges of its own tiles: row
counts around the edges of a tile, a half tile and a workgroup, running maxima raised inside the pipelined loop, block
lists of every block size (256: two workgroups share a row block), gather and scatter."""
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


@pytest.mark.parametrize("Hq,Hkv,Lc,d,window,Bs,form", [
    (4, 4, 8192, 128, 512, 128, 2),      # 256 workgroups of 128 rows: all at once, split keys
    (4, 2, 8193, 64, 512, 128, 3),       # one more tile of rows per head: two rounds, four wavefronts
    (12, 4, 4096, 64, 1024, 256, 3),     # 384 workgroups
    (2, 2, 4096, 128, 512, 64, 3),       # blocks of 64: four wavefronts whatever their number
    (2, 2, 4096, 64, 512, 256, 2),
])
def test_form_taken_under_a_block_list(tsa, Hq, Hkv, Lc, d, window, Bs, form):
    """Which form a launch with a block list takes, seen in the bits of its output: the split form merges two sums per row at
    the end and rounds differently (the two others often agree in every bit)."""
    r = par._rng(1500 + Lc)
    Q, K, V = (par.gu.to_dev(par.gu.rand_bits(r, (1, h, Lc, d))) for h in (Hq, Hkv, Hkv))
    bl = par.orc.lambda_block_list(Lc, Bs, window, 1)
    desc = tsa.make_desc(1, Hq, Hkv, Lc, d, 1)
    ws = tsa.alloc_attend_workspace(desc, Lc, Hkv, par.gu.DEV)
    out = {}
    try:
        for f in (0, 2, 3):
            tsa.tsa_bench_set_attend_form(f)
            out[f] = par.torch.empty_like(Q)
            tsa.tsa_attend(desc, Q, K, V, Lc, Hkv, out[f], ws, block_list=par.torch.from_numpy(bl).to(par.gu.DEV), block_size=Bs,
                           max_blocks_per_row=bl.shape[1])
    finally:
        tsa.tsa_bench_set_attend_form(0)
    assert not par.torch.equal(out[2], out[3])
    assert par.torch.equal(out[0], out[form])


@pytest.mark.parametrize("Hq,Hkv,Lc,d,form", [(4, 4, 18900, 128, 2), (4, 2, 22600, 64, 3), (16, 2, 4090, 64, 2), (16, 2, 4300, 64, 3), (40, 8, 1300, 128, 3),
                                              (40, 8, 1000, 64, 2), (32, 8, 1792, 64, 2), (32, 8, 1793, 64, 3)])
def test_form_taken_without_a_list(tsa, Hq, Hkv, Lc, d, form):
    """Both sides of the line between the split form and four wavefronts, which rises with the number of heads; tsa_forward's
    launch takes the same side."""
    r = par._rng(1600 + Lc)
    torch = par.torch
    Q, K, V = (torch.from_numpy(r.standard_normal((1, h, Lc, d), dtype="float32")).to(par.gu.DEV).bfloat16() for h in (Hq, Hkv, Hkv))
    desc = tsa.make_desc(1, Hq, Hkv, Lc, d, 1)
    ws = tsa.alloc_attend_workspace(desc, Lc, Hkv, par.gu.DEV)
    idx = torch.arange(Lc, dtype=torch.int32, device=par.gu.DEV).repeat(1, Hq, 1)
    Vt = tsa.alloc_attend_workspace(desc, Lc, Hq, par.gu.DEV)
    tsa.tsa_compress_v_tiles(desc, V, idx, Lc, Vt)
    out, fused = {}, {}
    try:
        for f in (0, 2, 3):
            tsa.tsa_bench_set_attend_form(f)
            out[f], fused[f] = torch.empty_like(Q), torch.empty_like(Q)
            tsa.tsa_attend(desc, Q, K, V, Lc, Hkv, out[f], ws)
            tsa.tsa_attend_fused(desc, Q, K, Vt, idx, idx, Lc, O=fused[f])
    finally:
        tsa.tsa_bench_set_attend_form(0)
    assert not torch.equal(out[2], out[3])
    assert torch.equal(out[0], out[form]) and torch.equal(fused[0], out[0])
