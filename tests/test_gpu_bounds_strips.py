"""Bound estimators at the orders where the strips of the matrix-vector product change length,
with ragged last tiles and a row stride beyond the order, against the CPU oracle (the same
recurrence in FP64, only summation orders differ: 1e-9 of the spectral width)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import bounds  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def snf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf as s
    s.lib()
    return s


def _sym(n, rng):
    a = rng.standard_normal((n, n)) / np.sqrt(2.0 * n)
    return a + a.T


@pytest.mark.parametrize("n", [1, 64, 65, 1985, 2049, 3009, 3201])
def test_strips_match_oracle(snf, n):
    rng = np.random.default_rng(n)
    f, d, v0, steps = _sym(n, rng), 0.3 * _sym(n, rng), rng.standard_normal(n), 5
    wide = torch.full((2, n, n + 3), 7.0, device="cuda:0", dtype=torch.float64)
    wide[0, :, :n], wide[1, :, :n] = torch.tensor(f), torch.tensor(d)
    F, D = wide[0, :, :n], wide[1, :, :n]
    v = torch.tensor(v0, device="cuda:0")
    got = snf.spectral_bounds(F, steps, start=v)
    want = bounds.spectral_bounds(f, v0, steps) + bounds.gershgorin(f)
    scale = max(4.0, want[3] - want[2])
    assert np.max(np.abs(np.array(got) - np.array(want))) <= 1e-9 * scale
    if n > steps:
        got = snf.gap_bounds(F, D, -2.0, 2.0, steps, start=v)
        assert np.max(np.abs(np.array(got) - bounds.gap_bounds(f, d, -2.0, 2.0, v0, steps))) <= 4e-9
