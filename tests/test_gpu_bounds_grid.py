"""Bound estimators at the orders where the strips of the matrix-vector product get three, four and
five tiles, and where the strips of a row number a multiple of 8, against the CPU oracle (the same
recurrence in FP64, only summation orders differ: 1e-9 of the spectral width)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import bounds  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3264, 3265, 4544, 4545, 8000, 12737])
def test_orders_match_oracle(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    g = torch.Generator(device="cuda:0").manual_seed(n)
    F = torch.randn(n, n, generator=g, device="cuda:0", dtype=torch.float64).div_((2.0 * n) ** 0.5)
    F = F + F.T
    D = F.flip(0, 1).mul_(0.3).contiguous()
    v = torch.randn(n, generator=g, device="cuda:0", dtype=torch.float64)
    f, d, v0, steps = F.cpu().numpy(), D.cpu().numpy(), v.cpu().numpy(), 3
    got = snf.spectral_bounds(F, steps, start=v)
    want = bounds.spectral_bounds(f, v0, steps) + bounds.gershgorin(f)
    assert np.max(np.abs(np.array(got) - np.array(want))) <= 1e-9 * max(4.0, want[3] - want[2])
    got = snf.gap_bounds(F, D, -2.0, 2.0, steps, start=v)
    assert np.max(np.abs(np.array(got) - bounds.gap_bounds(f, d, -2.0, 2.0, v0, steps))) <= 4e-9
