"""Scoring around 33 to 64 chunks of up to 384 keys with four or more heads per KV head, where workgroups may take fewer heads on
chunks twice as long (which calls do: test_score_plan.py)."""
import pytest

from tests import test_gpu_parity as par

pytestmark = pytest.mark.gpu

tsa = par.tsa


@pytest.mark.parametrize("B,Hq,Hkv,L,d,Lq", [
    (1, 4, 1, 8192, 64, 33), (1, 4, 1, 8193, 64, 33),         # 32 and 33 chunks of 256 keys
    (1, 5, 1, 8449, 64, 20), (1, 3, 1, 8449, 64, 20),         # a third round of heads with one idle slot; a group of three
    (1, 8, 2, 16384, 64, 9), (1, 8, 2, 16385, 64, 9),         # 64 and 65 chunks
    (2, 4, 1, 9000, 128, 70),
    (1, 8, 1, 8449, 64, 40), (1, 10, 2, 8193, 128, 100), (2, 20, 4, 9000, 64, 20)])      # twice as long: one head, two sets, idle slots
def test_score(tsa, B, Hq, Hkv, L, d, Lq):
    par.test_score(tsa, B, Hq, Hkv, L, d, Lq)
