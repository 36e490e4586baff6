"""FP64 solves of small and middle order (one workgroup, or a tile per compute unit) at the
orders where the tile, the number of k-steps or the LDS layout changes, against the exact
projector of a rotated spectrum at the FP64 parity tolerance 1e-8 sqrt(n); the result is exactly
symmetric, and a row stride beyond n is left alone."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def snf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf as s
    s.lib()
    return s


def _case(n, n_occ, mu, gap):
    g = torch.Generator(device="cuda:0").manual_seed(n)
    q, _ = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda:0", dtype=torch.float64))
    lam = torch.cat([torch.linspace(-1.0, mu - gap / 2, n_occ, dtype=torch.float64),
                     torch.linspace(mu + gap / 2, 1.0, n - n_occ, dtype=torch.float64)]).cuda()
    f = (q * lam) @ q.T
    return (f + f.T) / 2, q[:, :n_occ] @ q[:, :n_occ].T


def _solve(snf, n, scheme, **kw):
    n_occ, mu, gap = max(1, min(n - 1, int(0.55 * n))), 0.1, 0.05
    f, ref = _case(n, n_occ, mu, gap)
    wide = torch.full((n, n + 3), 7.0, device="cuda:0", dtype=torch.float64)
    wide[:, :n] = f
    d = torch.full((n, n + 3), 7.0, device="cuda:0", dtype=torch.float64)
    d, r = snf.purify_dense(wide[:, :n], scheme, "fp64", out=d[:, :n], lambda_min=-1.0,
                            lambda_max=1.0, homo=mu - gap / 2, lumo=mu + gap / 2, mu=mu, xi=gap,
                            n_occ=n_occ, tol=1e-9, max_iter=100, **kw)
    assert r["status"] == "ok", r["status"]
    assert r["device_ms"] > 0.0 and r["log"][-1]["e"] == r["idem_err"] <= 1e-9
    err = float(torch.linalg.norm(d - ref))
    print(f"n={n} {scheme}: {r['products']} products, |D - D_exact|_F = {err:.2e}")
    assert err <= 1e-8 * math.sqrt(n)
    assert torch.equal(d, d.T)
    assert bool((d._base[:, n:] == 7.0).all())
    return r


EDGES = [2, 3, 16, 17, 32, 33, 64, 65, 96, 97, 127, 128, 129, 255, 256, 513, 704, 705, 768, 1024,
         1056, 1057, 1408, 1409, 1760, 1761, 2048, 2112, 2113]


@pytest.mark.parametrize("n", EDGES)
def test_one_product_schemes(snf, n):
    _solve(snf, n, "snf_varmu")
    _solve(snf, n, "sp2")


@pytest.mark.parametrize("n", EDGES)
def test_chains_of_products(snf, n):
    _solve(snf, n, "snf_fixmu")
    if n in (3, 64, 65, 80, 128, 129, 705, 1057, 1409, 1761, 2112):
        _solve(snf, n, "snf_fixmu3")
        _solve(snf, n, "snf_pij", poly_ij=(3, 1))
        _solve(snf, n, "snf_pij", poly_ij=(5, 3))


@pytest.mark.parametrize("n", [40, 100, 300])
def test_stops(snf, n):
    """Too few iterations, a non-finite input and the wrong occupation end as they should."""
    f, _ = _case(n, n // 2, 0.0, 0.1)
    kw = dict(lambda_min=-1.0, lambda_max=1.0, homo=-0.05, lumo=0.05, n_occ=n // 2, tol=1e-10)
    _, r = snf.purify_dense(f, "snf_varmu", max_iter=3, **kw)
    assert r["status"] == "noconv" and r["iterations"] == 3 and r["products"] == 4
    bad = f.clone()
    bad[1, 2] = bad[2, 1] = math.nan
    _, r = snf.purify_dense(bad, "snf_varmu", max_iter=50, **kw)
    assert r["status"] == "nonfinite" and r["products"] == 1
    _, r = snf.purify_dense(f, "snf_varmu", max_iter=50, **dict(kw, n_occ=n // 2 - 2))
    assert r["status"] == "mixed"
