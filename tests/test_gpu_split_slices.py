"""Stand-alone products whose tiles are all cut into k-slices, some, or none (ragged orders beside
the edges of the tiles), against FP64 products of the operands rounded as the kernel rounds them:
an accumulation in the product's precision over k in slices, so each entry is within
2 n u |A| |B| of it (u of FP64 or FP32), after the storing of Y in FP64."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ROUND = {"fp64": lambda t: t, "fp32": lambda t: t.float().double(),
         "bf16_ref64": lambda t: t.float().bfloat16().double()}


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16_ref64"])
@pytest.mark.parametrize("n", [1, 127, 129, 640, 1025, 2048, 2177])
def test_products(n, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    g = torch.Generator(device="cuda:0").manual_seed(n)
    a = torch.randn(n, n, generator=g, device="cuda:0", dtype=torch.float64)
    b = torch.randn(n, n, generator=g, device="cuda:0", dtype=torch.float64)
    a, b = ((a + a.T) / 2).contiguous(), ((b + b.T) / 2).contiguous()
    u = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    for x, y in ((a, a), (a, b)):
        got = snf.step_dense(x, y, 1.0, 0.0, 0.0, prec)[0]
        rx, ry = ROUND[prec](x), ROUND[prec](y)
        ref = rx @ ry
        bound = 2.0 * n * (u + 2.0 ** -53) * (rx.abs() @ ry.abs()) + 1e-300
        assert bool(((got - ref).abs() <= bound).all())
        if x is y:
            assert torch.equal(got, got.T)
