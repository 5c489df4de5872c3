"""Scoring where workgroups take two heads on chunks twice as long (33 to 64 chunks of up to 384 keys, four or more heads per KV head),
and just outside of that range."""
import pytest

from tests import test_gpu_parity as par

pytestmark = pytest.mark.gpu

tsa = par.tsa


@pytest.mark.parametrize("B,Hq,Hkv,L,d,Lq", [
    (1, 4, 1, 8192, 64, 33), (1, 4, 1, 8193, 64, 33),         # 32 and 33 chunks of 256 keys
    (1, 5, 1, 8449, 64, 20), (1, 3, 1, 8449, 64, 20),         # a third round of heads with one idle slot; a group of three
    (1, 8, 2, 16384, 64, 9), (1, 8, 2, 16385, 64, 9),         # 64 and 65 chunks
    (2, 4, 1, 9000, 128, 70)])
def test_score(tsa, B, Hq, Hkv, L, d, Lq):
    par.test_score(tsa, B, Hq, Hkv, L, d, Lq)
