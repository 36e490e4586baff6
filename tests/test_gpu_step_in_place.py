"""A stand-alone step on matrices that already have the padded layout (read and written in
place) gives the same bits as on copies whose row stride, alignment or overlap rules that out."""
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


def _strided(a, ld, shift=0):
    n = a.shape[0]
    flat = torch.full((n * ld + shift,), 7.0, device="cuda:0", dtype=torch.float64)
    v = flat[shift:].view(n, ld)[:, :n]
    v.copy_(a)
    return v


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16_ref64"])
@pytest.mark.parametrize("n", [128, 129, 255, 256, 640, 1023])
@pytest.mark.parametrize("square", [True, False])
def test_same_bits(snf, prec, n, square):
    g = torch.Generator().manual_seed(n)
    a, b = (torch.randn(n, n, generator=g, dtype=torch.float64) / n ** 0.5 for _ in range(2))
    a, b = (a + a.T).cuda(), (b + b.T).cuda()
    b = a if square else b
    c = (-1.3, 2.1, 0.4)
    y, sums, _ = snf.step_dense(a, b, *c, prec)
    for ld, shift in ((n + 1, 0), (n + 2, 0), (n, 1)):
        sa = _strided(a, ld, shift)
        sb = sa if square else _strided(b, ld, shift)
        out = _strided(torch.zeros_like(a), ld, shift)
        y2, sums2, _ = snf.step_dense(sa, sb, *c, prec, out=out)
        assert torch.equal(y, y2) and sums == sums2
        flat = out._base if out._base is not None else out
        assert int((flat == 7.0).sum()) == flat.numel() - n * n     # nothing else was written
    # the result over the tail of the operand's memory: through a copy
    if n % 128 == 0 and square:
        flat = torch.empty(n * n + n, device="cuda:0", dtype=torch.float64)
        va, vy = flat[:n * n].view(n, n), flat[n:].view(n, n)
        va.copy_(a)
        y3, sums3, _ = snf.step_dense(va, va, *c, prec, out=vy)
        assert torch.equal(y, y3) and sums == sums3
