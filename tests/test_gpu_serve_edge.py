"""Served requests on both sides of the order where their products' tiles change (64x64 up to a
padded order of 2048, 128x128 beyond), against the exact projector of a diagonal-plus-rotation
spectrum and, bit for bit, alone against in a mix."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GAP = 0.1
MIX = [(2047, "snf_varmu", "fp64", {}), (2048, "snf_varmu", "fp32_ref64", {}),
       (2048, "snf_pij", "fp64", dict(poly_ij=(3, 1))), (2049, "snf_varmu", "fp64", {}),
       (2049, "snf_fixmu", "fp32_ref64", {}), (2176, "snf_pij", "fp64", dict(poly_ij=(3, 1)))]


def _case(n):
    k = n // 2
    g = torch.Generator(device="cuda:0").manual_seed(n)
    u = torch.randn(n, generator=g, device="cuda:0", dtype=torch.float64)
    u /= torch.linalg.norm(u)
    q = torch.eye(n, device="cuda:0", dtype=torch.float64) - 2.0 * torch.outer(u, u)   # a reflection
    lam = torch.cat([torch.linspace(-1.0, -GAP / 2, k, dtype=torch.float64),
                     torch.linspace(GAP / 2, 1.0, n - k, dtype=torch.float64)]).cuda()
    f = (q * lam) @ q.T
    kw = dict(lambda_min=-1.0, lambda_max=1.0, homo=-GAP / 2, lumo=GAP / 2, mu=0.0, xi=GAP,
              n_occ=k, tol=1e-9, max_iter=100)
    return ((f + f.T) / 2).contiguous(), q[:, :k] @ q[:, :k].T, kw


def test_both_sides_of_the_limit():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    cases = [_case(n) for n, *_ in MIX]
    with snf.Server(4 << 30, max_slots=16) as sv:
        tickets = [sv.submit_device(f, s, p, **kw, **more)
                   for (f, _, kw), (_, s, p, more) in zip(cases, MIX)]
        mixed = [sv.wait(t) for t in tickets]
        alone = [sv.wait(sv.submit_device(f, s, p, **kw, **more))
                 for (f, _, kw), (_, s, p, more) in zip(cases, MIX)]
    torch.cuda.synchronize()
    for (n, scheme, prec, _), (_, ref, _), (d, r), (d1, r1) in zip(MIX, cases, mixed, alone):
        assert r["status"] == r1["status"] == "ok", (n, scheme, prec, r["status"])
        # FP64: the parity bar; FP32 start: 2^-24 sqrt(n) for each of at most 10 steps, over the gap
        tol = 1e-8 if prec == "fp64" else 10 * 2.0 ** -24 / GAP
        assert float(torch.linalg.norm(d - ref)) <= tol * math.sqrt(n), (n, scheme, prec)
        assert torch.equal(d, d.T) and torch.equal(d, d1)
        assert r["products"] == r1["products"] and r["idem_err"] == r1["idem_err"]
