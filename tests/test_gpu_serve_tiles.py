"""Served requests at the orders where their products' tiles change (64x64 up to a padded order of
2816, 128x128 beyond), against the exact projector of a rotated spectrum: FP64 within the parity
tolerance 1e-8 sqrt(n); FP32 start with FP64 end within 2^-24 sqrt(n) for each of at most 10 FP32
steps, turned by at most 1 / gap.  All at once on one server and each alone give the same bits."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GAP = 0.05
MIX = [(2, "snf_varmu", "fp64", {}), (63, "sp2", "fp64", {}), (64, "snf_varmu", "fp32_ref64", {}),
       (65, "snf_fixmu", "fp64", {}), (127, "snf_varmu", "fp32_ref64", {}),
       (129, "snf_pij", "fp64", dict(poly_ij=(3, 1))), (192, "sp2", "fp32_ref64", {}),
       (193, "snf_fixmu3", "fp64", {}), (512, "snf_varmu", "fp64", {}),
       (513, "snf_varmu", "fp32_ref64", {}), (2816, "snf_varmu", "fp32_ref64", {}),
       (2816, "snf_fixmu", "fp64", {}), (2817, "snf_varmu", "fp32_ref64", {}),
       (2817, "snf_pij", "fp64", dict(poly_ij=(3, 1)))]


def _case(n):
    n_occ, mu = max(1, min(n - 1, int(0.55 * n))), 0.1
    g = torch.Generator(device="cuda:0").manual_seed(n)
    q, _ = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda:0", dtype=torch.float64))
    lam = torch.cat([torch.linspace(-1.0, mu - GAP / 2, n_occ, dtype=torch.float64),
                     torch.linspace(mu + GAP / 2, 1.0, n - n_occ, dtype=torch.float64)]).cuda()
    f = (q * lam) @ q.T
    kw = dict(lambda_min=-1.0, lambda_max=1.0, homo=mu - GAP / 2, lumo=mu + GAP / 2, mu=mu, xi=GAP,
              n_occ=n_occ, tol=1e-9, max_iter=100)
    return ((f + f.T) / 2).contiguous(), q[:, :n_occ] @ q[:, :n_occ].T, kw


def test_tiles_of_a_mix():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    cases = [_case(n) for n, *_ in MIX]
    with snf.Server(4 << 30, max_slots=32) as sv:
        tickets = [sv.submit_device(f, s, p, **kw, **more)
                   for (f, _, kw), (_, s, p, more) in zip(cases, MIX)]
        mixed = [sv.wait(t) for t in tickets]
        alone = [sv.wait(sv.submit_device(f, s, p, **kw, **more))
                 for (f, _, kw), (_, s, p, more) in zip(cases, MIX)]
    torch.cuda.synchronize()
    for (n, scheme, prec, _), (_, ref, _), (d, r), (d1, r1) in zip(MIX, cases, mixed, alone):
        assert r["status"] == r1["status"] == "ok", (n, scheme, prec, r["status"])
        err = float(torch.linalg.norm(d - ref))
        print(f"n={n} {scheme} {prec}: {r['products']} products, |D - D_exact|_F = {err:.2e}")
        tol = 1e-8 if prec == "fp64" else 10 * 2.0 ** -24 / GAP
        assert err <= tol * math.sqrt(n)
        assert torch.equal(d, d.T) and torch.equal(d, d1)
        assert all(r[k] == r1[k] for k in ("products", "iterations", "branches", "idem_err"))
        assert len(r["branches"]) == r["iterations"] and r["idem_err"] <= 1e-9
