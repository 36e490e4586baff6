"""The scaling of the P_{i,j} schemes, whose two Eq. 3 the halves of a wave solve side by side, in
the one-workgroup solve, the direct steps and the schedule kernel: bit for bit that of plain
bisections in double precision along the recurrence of both bounds."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _poly(i, j, x):
    y, acc = 1.0 - x, 0.0
    for k in range(j, -1, -1):
        acc = acc * y + float(math.comb(i + k, k))
    xp = x
    for _ in range(i):
        xp = xp * x
    return xp * acc


def _bisect(lo, hi, below):
    while True:
        mid = 0.5 * (lo + hi)
        if mid <= lo or mid >= hi:
            return lo
        g = below(mid)
        if g is None:
            return mid
        if g:
            lo = mid
        else:
            hi = mid


def _xstar(i, j):
    def below(x):
        g = _poly(i, j, x) - x
        return None if g == 0.0 else g < 0.0
    return _bisect(0.0, 1.0, below)


def _side(i, j, xs, a):
    """The root of one side's Eq. 3."""
    if not 0.0 < a < xs:
        return 1.0
    return _bisect(1.0, xs / (xs - a), lambda v: _poly(i, j, xs * (1.0 - v)) -
                   _poly(i, j, xs - v * (xs - a)) < 0.0)


def _next(i, j, xs, a, v):
    return max(_poly(i, j, xs * (1.0 - v)), _poly(i, j, xs - v * (xs - a)))


@pytest.mark.parametrize("n", [3, 64, 100, 2200])
@pytest.mark.parametrize("i,j", [(3, 1), (1, 3), (5, 3), (1, 5), (3, 3)])
@pytest.mark.parametrize("gap", [0.4, 1e-3, 1e-9])
def test_alpha_bits(n, i, j, gap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    mu = -0.5
    k = max(1, n // 2)
    lam = torch.ones(n, dtype=torch.float64, device="cuda:0")
    lam[:k] = -1.0
    lam[0], lam[n - 1] = mu - gap / 2, mu + gap / 2
    _, r = snf.purify_dense(torch.diag(lam).contiguous(), "snf_pij", "fp64", lambda_min=-1.0,
                            lambda_max=1.0, mu=mu, xi=gap, n_occ=k, tol=1e-10, max_iter=100,
                            poly_ij=(i, j))
    assert r["status"] == "ok", r["status"]
    steps = [rec for rec in r["log"] if rec["branch"] is not None]
    xs = _xstar(i, j)
    gamma = max((mu + 1.0) / (1.0 - xs), (1.0 - mu) / xs)
    a, b = xs - gap / (2.0 * gamma), (1.0 - xs) - gap / (2.0 * gamma)
    other = 0
    for rec in steps:
        assert rec["beta"] == a and rec["betabar"] == 1.0 - b, rec
        lo, hi = _side(i, j, xs, a), _side(j, i, 1.0 - xs, b)
        assert rec["alpha"] == min(lo, hi), rec
        other += lo != hi
        a, b = _next(i, j, xs, a, rec["alpha"]), _next(j, i, 1.0 - xs, b, rec["alpha"])
    assert steps and any(rec["alpha"] > 1.0 for rec in steps)
    assert other or i == j                      # the two sides' equations differ
