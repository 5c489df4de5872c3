"""Block lists of more than 64 entries per row: the entries are counted 64 at a time, up to the first one outside 0..qb."""
import numpy as np
import pytest

from tests import test_gpu_parity as par

pytestmark = pytest.mark.gpu

tsa = par.tsa


@pytest.mark.parametrize("form", [1, 2, 3])
@pytest.mark.parametrize("d,Lc,end", [(64, 64 * 67 - 5, -1), (128, 64 * 66, 99), (64, 64 * 65, -1)])
def test_long_block_lists(tsa, form, d, Lc, end):
    r = par._rng(1700 + Lc)
    orc, gu, torch = par.orc, par.gu, par.torch
    nb = (Lc + 63) // 64
    Qb, Kb, Vb = (gu.rand_bits(r, (1, 2, Lc, d)) for _ in range(3))
    # row qb lists every block up to its own (1 to nb entries), then `end` (no block, or one beyond the row's own), then
    # entries that would be valid and must not be read as such
    bl = np.zeros((nb, nb + 2), dtype=np.int32)
    for qb in range(nb):
        bl[qb, :qb + 1] = np.arange(qb + 1)
        bl[qb, qb + 1] = end
    desc = tsa.make_desc(1, 2, 2, Lc, d, 1)
    O = torch.empty((1, 2, Lc, d), dtype=torch.bfloat16, device=gu.DEV)
    tsa.tsa_bench_set_attend_form(form)
    try:
        tsa.tsa_attend(desc, gu.to_dev(Qb), gu.to_dev(Kb), gu.to_dev(Vb), Lc, 2, O, tsa.alloc_attend_workspace(desc, Lc, 2, gu.DEV),
                       block_list=torch.from_numpy(bl).to(gu.DEV), block_size=64, max_blocks_per_row=bl.shape[1])
        torch.cuda.synchronize()
    finally:
        tsa.tsa_bench_set_attend_form(0)
    # the lists together are plain causal attention
    want = orc.attend(orc.bf16_to_f64(Qb), orc.bf16_to_f64(Kb), orc.bf16_to_f64(Vb))
    gu.assert_output_close(gu.from_dev(O), orc.f64_to_bf16(want), "attend(long block lists)")
