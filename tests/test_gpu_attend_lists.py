"""Which form of the attention kernel a launch takes under a block list with room for every block of the set: the one its
longest chain asks for, as without a list; seen in the bits of its output (the split form merges two sums per row at the end
and rounds differently), in tsa_attend and in the fused launch alike."""
import pytest

from tests import test_gpu_parity as par

pytestmark = pytest.mark.gpu

tsa = par.tsa


@pytest.mark.parametrize("Hq,Hkv,Lc,d,window,Bs,form", [
    (12, 4, 4096, 128, 4096, 128, 2),    # the list's row has room for all blocks
    (12, 4, 4095, 64, 4095, 64, 2),      # a ragged last block, blocks of 64
    (12, 4, 4097, 128, 3584, 256, 3),    # one block short of it
    (28, 4, 2048, 64, 2048, 128, 3),     # ratio 2.03, below the line
    (28, 4, 1500, 64, 1500, 256, 2),
])
def test_form_taken_under_a_list_as_long_as_the_set(tsa, Hq, Hkv, Lc, d, window, Bs, form):
    r = par._rng(1700 + Lc)
    torch = par.torch
    Q, K, V = (torch.from_numpy(r.standard_normal((1, h, Lc, d), dtype="float32")).to(par.gu.DEV).bfloat16() for h in (Hq, Hkv, Hkv))
    bl = par.orc.lambda_block_list(Lc, Bs, window, 1)
    assert (bl.shape[1] * Bs >= Lc) == (window != 3584)
    kw = dict(block_list=torch.from_numpy(bl).to(par.gu.DEV), block_size=Bs, max_blocks_per_row=bl.shape[1])
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
            tsa.tsa_attend(desc, Q, K, V, Lc, Hkv, out[f], ws, **kw)
            tsa.tsa_attend_fused(desc, Q, K, Vt, idx, idx, Lc, O=fused[f], **kw)
    finally:
        tsa.tsa_bench_set_attend_form(0)
    assert not torch.equal(out[2], out[3])
    assert torch.equal(out[0], out[form]) and torch.equal(fused[0], out[0])
