"""More than 64 scoring queries: two sets of them, whose column sums meet in LDS two tiles later.  Chunks of one tile and a few,
with and without masked tiles, every number of heads per workgroup, idle slots."""
import pytest

from tests import test_gpu_parity as par

pytestmark = pytest.mark.gpu

tsa = par.tsa


@pytest.mark.parametrize("B,Hq,Hkv,L,d,Lq", [
    (1, 1, 1, 65, 64, 65), (1, 4, 2, 128, 128, 128), (1, 3, 1, 129, 64, 100), (2, 5, 1, 300, 128, 96), (1, 4, 1, 700, 64, 127),
    (1, 8, 8, 2000, 128, 70), (1, 10, 1, 5001, 64, 128), (3, 6, 2, 4097, 128, 66), (1, 32, 8, 33000, 64, 100)])
def test_score(tsa, B, Hq, Hkv, L, d, Lq):
    par.test_score(tsa, B, Hq, Hkv, L, d, Lq)
