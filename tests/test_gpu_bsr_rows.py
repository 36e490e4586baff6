"""One block-sparse step on block-tridiagonal matrices whose rows hold few, many and more than 256
bitmap words: the pattern is exactly block-pentadiagonal, the blocks match FP64 products of the
FP32 blocks to the FP32 accumulation bound of 96 terms, and the sums match the blocks."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
B = 32


@pytest.fixture(scope="module")
def snf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf as s
    s.lib()
    return s


@pytest.mark.parametrize("nb", [5, 40, 1100, 8300])
@pytest.mark.parametrize("screen", [0.0, 1e-30])
def test_block_tridiagonal(snf, nb, screen):
    g = torch.Generator(device="cuda:0").manual_seed(nb)
    d = torch.randn(nb, B, B, generator=g, device="cuda:0") / 16
    d = (d + d.transpose(1, 2)) / 2
    o = torch.randn(nb - 1, B, B, generator=g, device="cuda:0") / 16      # (I, I + 1)
    rows, cols, vals = [], [], torch.zeros(3 * nb - 2, B, B, device="cuda:0")
    idx = {}
    for off in (-1, 0, 1):
        r = np.arange(max(0, -off), min(nb, nb - off))
        rows.append(r)
        cols.append(r + off)
    r, c = np.concatenate(rows), np.concatenate(cols)
    order = np.lexsort((c, r))
    r, c = r[order], c[order]
    rt, ct = torch.tensor(r).cuda(), torch.tensor(c).cuda()
    vals[rt == ct] = d
    vals[ct == rt + 1] = o
    vals[ct == rt - 1] = o.transpose(1, 2)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=nb))]).astype(np.int32)
    (rp, ci, va), sums, _ = snf.step_bsr(torch.tensor(ptr).cuda(),
                                         torch.tensor(c.astype(np.int32)).cuda(), vals, nb * B,
                                         1.0, 0.0, 0.0, screen_tau=screen)
    R = np.repeat(np.arange(nb), np.diff(rp.cpu().numpy()))
    C = ci.cpu().numpy()
    width = np.minimum(np.arange(nb) + 2, nb - 1) - np.maximum(np.arange(nb) - 2, 0) + 1
    assert np.array_equal(np.diff(rp.cpu().numpy()), width)
    assert np.array_equal(C - R, np.concatenate([np.arange(max(0, i - 2), min(nb - 1, i + 2) + 1) - i
                                                 for i in range(nb)]))
    dd, oo = d.double(), o.double()
    off = torch.tensor(C - R).cuda()
    z = torch.zeros(1, B, B, device="cuda:0", dtype=torch.float64)
    below, above = torch.cat([z, oo]), torch.cat([oo, z])      # (I - 1, I), (I, I + 1)
    mm = lambda x, y: torch.stack([a @ b for a, b in zip(x, y)]) if len(x) < 64 else torch.bmm(x, y)
    ref = {0: mm(dd, dd) + mm(below.transpose(1, 2).contiguous(), below) +
              mm(above, above.transpose(1, 2).contiguous()),
           1: mm(dd[:-1].contiguous(), oo) + mm(oo, dd[1:].contiguous()),
           2: mm(oo[:-1].contiguous(), oo[1:].contiguous())}
    bound = 96 * 2.0 ** -24 * 96 * float(vals.abs().max()) ** 2
    for k, want in ref.items():
        assert float((va[off == k].double() - want).abs().max()) <= bound
        assert torch.equal(va[off == -k], va[off == k].transpose(1, 2))
    tr = float(va[off == 0].double().diagonal(dim1=1, dim2=2).sum())
    fro = float((va.double() ** 2).sum())
    assert abs(sums[1] - tr) <= 1e-5 * nb and abs(sums[2] - fro) <= 1e-6 * fro
