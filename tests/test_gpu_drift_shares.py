"""The drift at the lines where the shares of the workgroups change (8192 and 16384 rows), and with a workspace that holds no more
partials than one per 64 rows."""
import numpy as np
import pytest
import torch

from tests import test_gpu_drift as drift

pytestmark = pytest.mark.gpu

tsa = drift.tsa


@pytest.mark.parametrize("n_tokens,width", [(15, 64), (17, 1032), (511, 64), (2047, 520), (8192, 64), (8193, 64), (16384, 64), (16385, 64), (40000, 16)])
def test_shares(tsa, n_tokens, width):
    orc, gu = drift.orc, drift.gu
    r = np.random.Generator(np.random.PCG64(880 + n_tokens))
    hin = gu.rand_bits(r, (n_tokens, width))
    hout = orc.f64_to_bf16(orc.bf16_to_f64(hin) + 0.3 * r.standard_normal((n_tokens, width)))
    a, b = gu.to_dev(hin), gu.to_dev(hout)
    want = orc.layer_drift(orc.bf16_to_f64(hin), orc.bf16_to_f64(hout), 1e-3)
    least = ((n_tokens + 63) // 64 * 8 + 255) // 256 * 256
    for ws in (None, torch.empty(least, dtype=torch.uint8, device=gu.DEV)):
        out = torch.full((1,), -1.0, dtype=torch.float32, device=gu.DEV)
        tsa.tsa_layer_drift(a, b, 1e-3, out, ws)
        assert abs(out.item() - want) <= 2e-6 * abs(want) + 1e-9          # fp32 sums of `width` squares


@pytest.mark.parametrize("n_tokens,width", [(2047, 64), (8192, 64), (20000, 16)])
def test_one_result_per_workspace_size(tsa, n_tokens, width):
    gu = drift.gu
    r = np.random.Generator(np.random.PCG64(890 + n_tokens))
    a, b = (gu.to_dev(gu.rand_bits(r, (n_tokens, width))) for _ in range(2))
    least = ((n_tokens + 63) // 64 * 8 + 255) // 256 * 256
    full = tsa.load_library().tsa_layer_drift_workspace_bytes(n_tokens)
    assert full > least
    got = {}
    for size in (full, least, least + 64, full + 4096, full, least):
        out = torch.full((1,), -1.0, dtype=torch.float32, device=gu.DEV)
        tsa.tsa_layer_drift(a, b, 1e-3, out, torch.empty(size, dtype=torch.uint8, device=gu.DEV))
        assert got.setdefault(min(size, full), out.item()) == out.item()      # room beyond the full size changes nothing
    with pytest.raises(tsa.TsaError):
        tsa.tsa_layer_drift(a, b, 1e-3, torch.empty(1, device=gu.DEV), torch.empty(least - 8, dtype=torch.uint8, device=gu.DEV))
