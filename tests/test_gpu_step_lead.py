"""Solves whose steps are several launches, enqueued a few steps ahead of the device: they end as
they should when the iteration limit lies below, at and above that lead, when the first state is
already the last, and when the limit is never reached; a limit cuts the same solve short."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(130, "fp32_ref64"), (2049, "fp32_ref64"),
                                    (300, "bf16_ref64"), (300, "fp32"), (2200, "fp64")])
def test_ends(n, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    g = torch.Generator(device="cuda:0").manual_seed(n)
    q, _ = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda:0", dtype=torch.float64))
    lam = torch.cat([torch.linspace(-1.0, -0.1, n // 2, dtype=torch.float64),
                     torch.linspace(0.1, 1.0, n - n // 2, dtype=torch.float64)]).cuda()
    f = (q * lam) @ q.T
    f = ((f + f.T) / 2).contiguous()
    kw = dict(lambda_min=-1.0, lambda_max=1.0, homo=-0.1, lumo=0.1, n_occ=n // 2, tol=1e-8)
    if prec == "bf16_ref64":
        kw["gap_switch"] = 0.5
    _, full = snf.purify_dense(f, "snf_varmu", prec, max_iter=100, **kw)
    assert full["status"] in ("ok", "ok_floor"), full["status"]
    assert len(full["log"]) == full["products"] == full["iterations"] + 1
    for limit in (1, 3, 4, 5):
        _, r = snf.purify_dense(f, "snf_varmu", prec, max_iter=limit, **kw)
        assert r["status"] == "noconv" and r["iterations"] == limit
        assert r["log"][:limit] == full["log"][:limit]
    bad = f.clone()
    bad[0, 1] = bad[1, 0] = math.nan
    _, r = snf.purify_dense(bad, "snf_varmu", prec, max_iter=100, **kw)
    assert r["status"] == "nonfinite"
    # a projector at the bounds: X_0 is the result, one product certifies it
    p = 1.0 - 2.0 * (torch.arange(n, device="cuda:0") < n // 2).double()
    kw.update(homo=-1.0, lumo=1.0)
    _, r = snf.purify_dense(torch.diag(p).contiguous(), "snf_varmu", prec, max_iter=100, **kw)
    assert r["status"] in ("ok", "ok_floor") and r["products"] <= 2
