"""How many terms a product of the FP64 solves adds to one running sum before partial sums are
added.  One step X -> X^2 on a matrix whose row pairs multiply to one term 1 and, everywhere else,
terms of 2^-55 (times 2^-10): added to a sum that holds the 1, such a term is lost, so what is
missing from the result counts the terms behind the 1 in its chain.  Tolerance: the longest chain
the kernels leave at that order, plus half a unit in the last place (4 terms) for each later
addition of a partial sum."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

PAIRS = 4


def _lost(snf, n):
    """Lost terms of the products of the PAIRS last row pairs, each with its 1 at another k."""
    m = n - 2 * PAIRS
    x = torch.zeros(n, n, dtype=torch.float64)
    x[torch.arange(m), torch.arange(m)] = 2.0 ** -7
    for p in range(PAIRS):
        a, b = m + 2 * p, m + 2 * p + 1
        x[a, :m], x[b, :m] = 2.0 ** -32, 2.0 ** -33
        x[a, p * m // PAIRS] = x[b, p * m // PAIRS] = 2.0 ** -5
        x[:m, a], x[:m, b] = x[a, :m], x[b, :m]
    f = (torch.eye(n, dtype=torch.float64) - x).cuda()
    # one squaring: ||X^2 - X||_F is 0.13 to 0.3 before it and below 0.01 behind it
    d, r = snf.purify_dense(f, "sp2", "fp64", lambda_min=0.0, lambda_max=1.0, n_occ=0, tol=0.1,
                            max_iter=5)
    assert r["status"] == "ok" and r["iterations"] == 1 and r["branches"] == "S", r
    d = d.cpu()
    return [(m - 1) - (float(d[m + 2 * p, m + 2 * p + 1]) * 2.0 ** 10 - 1.0) * 2.0 ** 55
            for p in range(PAIRS)]


@pytest.mark.parametrize("n,chain,adds", [
    (32, 8, 2), (64, 16, 2), (80, 20, 2),              # one workgroup: four chains
    (256, 256 // 16 + 8, 5), (400, 400 // 16 + 8, 5), (600, 600 // 16 + 8, 5),
    (704, 704 // 16 + 8, 5),                           # four chains a wave, four waves
    (705, 705 // 16 + 28, 7), (896, 896 // 16 + 28, 7), (1000, 1000 // 16 + 28, 7),
    (1056, 1056 // 16 + 28, 7),                        # four phases of whole load rounds (7 x 4)
    (1057, 1057 // 8 + 28, 5), (1152, 1152 // 8 + 28, 5)])
def test_chain_length(n, chain, adds):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    lost = _lost(snf, n)
    print(f"n={n}: {lost} terms lost")
    assert max(abs(v) for v in lost) <= chain - 1 + 4 * adds, lost
