"""The budget of rows that one workgroup takes in one launch (up to 16384 tokens), and the first row length beyond, where a chain of
launches takes over: against the oracle, and against each other on the same row.  One head, so that the summed scores are the
scores themselves and the count must be the oracle's."""
import numpy as np
import pytest

from tests import test_gpu_budget as bud

pytestmark = pytest.mark.gpu

tsa = bud.tsa

TAUS = (0.0, 1.23457e-5, 0.01234567, 0.3141593, 0.7654321, 1.0)     # (no multiples of a grid step: a tie would be decided by the last bit)


@pytest.mark.parametrize("L", [1, 2, 64, 65, 1023, 1025, 4096, 4097, 16383, 16384, 16385])
def test_row_lengths(tsa, L):
    r = np.random.Generator(np.random.PCG64(820 + L))
    few = r.integers(0, 5, size=(2, 1, L)) / 8.0                          # runs of equal scores, zeros among them
    grid = np.floor(r.random((2, 1, L)) ** 4 * 2.0 ** 20) / 2.0 ** 20     # masses on a grid: exact in any order
    crowd = np.where(r.random((2, 1, L)) < 0.97, 2.0 ** -10 + r.integers(0, 90, size=(2, 1, L)) * 2.0 ** -33, 4.0)   # one bin takes nearly all
    for s in (few, grid, crowd):
        s = s.astype(np.float32)
        s[:, 0, 0] = 1.0                                                   # (a total of zero has no answer)
        for tau in TAUS:
            got, want = bud._budget(tsa, s, tau), bud.orc.coverage_budget(s, tau)
            assert np.array_equal(got, want), (tau, got, want)


@pytest.mark.parametrize("L", [65, 4097, 16384])
def test_scores_over_many_binades(tsa, L):
    """Bins that hold two binades, bins below the smallest normal number; each threshold lies in the middle of a token's mass,
    far from where another order of the float64 additions would move the count."""
    r = np.random.Generator(np.random.PCG64(830 + L))
    s = np.ldexp(1.0 + r.random((1, 1, L)), r.integers(-140, 20, size=(1, 1, L))).astype(np.float32)
    asc = np.sort(s[0, 0].astype(np.float64))
    cum = np.cumsum(asc)
    for n in sorted({L - 1, L - 2, L - L // 20, L - L // 10}):
        tau = (cum[n - 1] - 0.5 * asc[n - 1]) / cum[-1]
        if tau <= 1e-12 or asc[n - 1] / cum[-1] < 1e-12:
            continue
        assert bud._budget(tsa, s, tau)[0] == L - n == bud.orc.coverage_budget(s, tau)[0]


@pytest.mark.parametrize("L", [2, 65, 4096, 4097, 16384])
def test_one_launch_and_the_chain_agree(tsa, L):
    """Tokens of score zero lie under every positive threshold: a row padded with them until the chain of launches takes it
    keeps the same number of tokens."""
    r = np.random.Generator(np.random.PCG64(840 + L))
    rows = [r.integers(0, 5, size=L) / 8.0,                                # runs of equal scores, zeros among them
            np.floor(r.random(L) ** 4 * 2.0 ** 20) / 2.0 ** 20,
            2.0 ** -10 + r.integers(0, 90, size=L) * 2.0 ** -33,           # one bin of the chain's first digit
            np.where(r.random(L) < 0.5, -0.0, 2.0 ** -149 * r.integers(0, 9, size=L))]     # below the smallest normal number
    rows.append(rows[1].copy())
    rows[-1][L // 2] = np.inf                                              # no answer in the definition, but one of them
    for i, row in enumerate(rows):
        s = row.astype(np.float32)
        s[0] = max(s[0], 2.0 ** -145) if i == 3 else 1.0
        padded = np.zeros(16385 + L % 7, dtype=np.float32)
        padded[:L] = s
        padded = r.permutation(padded)
        for tau in TAUS[1:]:
            got, want = bud._budget(tsa, s[None, None], tau), bud._budget(tsa, padded[None, None], tau)
            assert np.array_equal(got, want), (i, tau, got, want)
            if i < 3:
                assert np.array_equal(got, bud.orc.coverage_budget(s[None, None], tau)), (i, tau)
