"""snf_purify_dense_noalloc against snf_purify_dense where the solve runs in one workgroup (one,
two and four iterate buffers) and at the first orders of the direct steps: D bit for bit."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

from paper_1101_0265_amd import hamiltonians as H  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["snf_varmu", "sp2", "snf_fixmu", "snf_fixmu3"])
@pytest.mark.parametrize("n", [7, 40, 64, 80, 81])
def test_small_orders_match(scheme, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    h = H.random_spectrum_hamiltonian(n, n // 2, -1.0, -0.04, 0.04, 1.0, 100 + n)
    F = torch.tensor(h.F, device="cuda:0")
    p = snf.make_params(lambda_min=h.lambda_min, lambda_max=h.lambda_max, n_occ=h.n_occ,
                        homo=h.homo, lumo=h.lumo, mu=h.mu, xi=h.xi, tol=1e-10, max_iter=120)
    out = []
    for entry in ("snf_purify_dense_noalloc", "snf_purify_dense"):
        D = torch.full_like(F, 7.0)
        res = snf.Result()
        logs = (snf.LogRec * snf.LOG_MAX)()
        rc = getattr(snf.lib(), entry)(F.data_ptr(), n, n, ctypes.byref(p), snf.SCHEMES[scheme],
                                       snf.PRECISIONS["fp64"], D.data_ptr(), ctypes.byref(res),
                                       logs, snf.LOG_MAX, torch.cuda.current_stream().cuda_stream)
        assert rc == snf.OK, (entry, rc)
        out.append((D, snf.result_dict(res, logs)))
    (D_b, r_b), (D_a, r_a) = out
    assert torch.equal(D_b, D_a)
    assert r_b["log"] == r_a["log"] and r_b["idem_err"] == r_a["idem_err"]
    assert r_b["products"] == r_a["products"] and r_b["trace"] == r_a["trace"]
