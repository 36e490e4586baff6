"""Results of the Python entry points for operands that are column slices of wider matrices: the
library writes with the operand's row stride, so a result that the binding allocates must have it
and one that the caller gives must match."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,first", [(40, 0), (200, 0), (201, 0), (201, 1), (200, 3)])
def test_slices(n, first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    g = torch.Generator(device="cuda:0").manual_seed(n)
    q, _ = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda:0", dtype=torch.float64))
    k = n // 2
    lam = torch.cat([torch.linspace(-1.0, -0.1, k), torch.linspace(0.1, 1.0, n - k)])
    f = (q * lam.double().cuda()) @ q.T
    # (row strides and first columns of both parities: rows on any 8-byte address)
    wide = torch.zeros(n, 3 * n, device="cuda:0", dtype=torch.float64)
    wide[:, first:first + n] = (f + f.T) / 2
    F = wide[:, first:first + n]
    kw = dict(lambda_min=-1.0, lambda_max=1.0, homo=-0.1, lumo=0.1, n_occ=k, tol=1e-10)
    D, r = snf.purify_dense(F, "snf_varmu", **kw)
    assert D.stride() == F.stride() and D.untyped_storage().nbytes() >= 8 * ((n - 1) * 3 * n + n)
    assert r["status"] == "ok"
    assert float(torch.linalg.norm(D - q[:, :k] @ q[:, :k].T)) <= 1e-8 * math.sqrt(n)
    Y, _, _ = snf.step_dense(F, F, -1.0, 2.0, 0.0)
    assert Y.stride() == F.stride()
    ref = 2.0 * F - F.contiguous() @ F.contiguous()
    assert float(torch.linalg.norm(Y - ref)) <= 1e-12 * math.sqrt(n)
    B = torch.zeros_like(wide)[:, first:first + n]
    B.copy_(0.5 * F + torch.eye(n, device="cuda:0"))
    ref = -F.contiguous() @ B.contiguous() + 2.0 * F
    bound = {"fp64": 1e-12, "fp32": 1e-5, "bf16_ref64": 0.05}    # 8 units of the operands' rounding
    for precision, tol in bound.items():
        Y, _, _ = snf.step_dense(F, B, -1.0, 2.0, 0.0, precision)
        assert float(torch.linalg.norm(Y - ref)) <= tol * math.sqrt(n)
    small = torch.empty(n, n, device="cuda:0", dtype=torch.float64)
    with pytest.raises(ValueError):
        snf.purify_dense(F, "snf_varmu", out=small, **kw)
    with pytest.raises(ValueError):
        snf.step_dense(F, F, -1.0, 2.0, 0.0, out=small)
    with pytest.raises(ValueError):
        snf.purify_dense(F.contiguous(), "snf_varmu", out=small[:-1, :-1], **kw)
    with snf.Server(64 << 20, max_slots=2) as server, pytest.raises(ValueError):
        server.submit_device(F.contiguous(), out=F, **kw)
