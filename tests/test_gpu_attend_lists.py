"""Which form of the attention kernel a launch takes under a block list whose rows have room for more blocks than the window: the
split form while all of its workgroups run at once, never because of the room alone; seen in the bits of its output (the split
form merges two sums per row at the end and rounds differently), in tsa_attend and in the fused launch alike."""
import numpy as np
import pytest

from tests import test_gpu_parity as par

pytestmark = pytest.mark.gpu

tsa = par.tsa


@pytest.mark.parametrize("Hq,Hkv,Lc,d,window,Bs,form,tight_form", [
    (12, 4, 4096, 128, 4096, 128, 3, 3),    # 384 workgroups, every block listed
    (12, 4, 4095, 64, 4095, 64, 3, 3),      # a ragged last block, blocks of 64
    (12, 4, 4097, 128, 3584, 256, 3, 3),    # one block short of the whole set
    (28, 4, 2048, 64, 2048, 128, 3, 3),
    (28, 4, 1500, 64, 1500, 256, 3, 3),
    (16, 4, 4096, 128, 2048, 128, 3, 3),    # 512, a window of half the set
    (12, 4, 4096, 64, 512, 64, 3, 3),
    (12, 4, 2048, 128, 2048, 64, 2, 2),     # 192
    (8, 4, 4096, 64, 256, 64, 2, 3),        # 256: blocks of 64 in narrow rows keep four wavefronts
    (8, 4, 4097, 64, 256, 64, 3, 3),        # 264
    (12, 4, 2600, 64, 512, 64, 3, 3),       # 252 in a grid of 264
    (12, 4, 2600, 64, 512, 128, 2, 2),
])
def test_form_taken_under_a_list(tsa, Hq, Hkv, Lc, d, window, Bs, form, tight_form):
    r = par._rng(1700 + Lc)
    torch = par.torch
    Q, K, V = (torch.from_numpy(r.standard_normal((1, h, Lc, d), dtype="float32")).to(par.gu.DEV).bfloat16() for h in (Hq, Hkv, Hkv))
    tight = par.orc.lambda_block_list(Lc, Bs, window, 1)
    wide = np.full((tight.shape[0], (Lc + Bs - 1) // Bs + 1), -1, dtype=tight.dtype)     # the same lists, room for every block
    wide[:, :tight.shape[1]] = tight
    desc = tsa.make_desc(1, Hq, Hkv, Lc, d, 1)
    ws = tsa.alloc_attend_workspace(desc, Lc, Hkv, par.gu.DEV)
    idx = torch.arange(Lc, dtype=torch.int32, device=par.gu.DEV).repeat(1, Hq, 1)
    Vt = tsa.alloc_attend_workspace(desc, Lc, Hq, par.gu.DEV)
    tsa.tsa_compress_v_tiles(desc, V, idx, Lc, Vt)

    def both(bl, f):
        kw = dict(block_list=torch.from_numpy(bl).to(par.gu.DEV), block_size=Bs, max_blocks_per_row=bl.shape[1])
        plain, fused = torch.empty_like(Q), torch.empty_like(Q)
        tsa.tsa_bench_set_attend_form(f)
        try:
            tsa.tsa_attend(desc, Q, K, V, Lc, Hkv, plain, ws, **kw)
            tsa.tsa_attend_fused(desc, Q, K, Vt, idx, idx, Lc, O=fused, **kw)
        finally:
            tsa.tsa_bench_set_attend_form(0)
        return plain, fused

    of_form = {f: both(tight, f)[0] for f in (2, 3)}
    assert not torch.equal(of_form[2], of_form[3])
    for bl, f in ((tight, tight_form), (wide, form)):
        for got in both(bl, 0):
            assert torch.equal(got, of_form[f])
