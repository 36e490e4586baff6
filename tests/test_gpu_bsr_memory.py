"""A very sparse block matrix of large order: the device memory of a block-sparse step follows the
stored blocks and the lookup tables, with nothing that grows with the square of the block rows
beyond those (one word per super-tile pair would be 335 MB here)."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def test_memory_of_a_diagonal_matrix():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1101_0265_amd import snf
    nb = 32768
    rp = torch.arange(nb + 1, dtype=torch.int32, device="cuda:0")
    ci = torch.arange(nb, dtype=torch.int32, device="cuda:0")
    va = (0.5 * torch.eye(32, device="cuda:0")).expand(nb, 32, 32).contiguous()
    torch.cuda.synchronize()
    snf.lib().snf_shutdown()
    torch.cuda.empty_cache()
    free0, held0 = torch.cuda.mem_get_info()[0], torch.cuda.memory_reserved()
    (row_ptr, col_idx, val), sums, _ = snf.step_bsr(rp, ci, va, 32 * nb, 1.0, 0.0, 0.0)
    torch.cuda.synchronize()
    used = free0 - torch.cuda.mem_get_info()[0] - (torch.cuda.memory_reserved() - held0)
    snf.lib().snf_shutdown()
    # values of X, the product and the result; bitmap and prefix counts of X and of the product;
    # arrays grow by a quarter; the lists and sums along the rows are below 10 MB
    blocks, tables = nb * 4096, nb * (nb // 32) * 4
    print(f"{used / 1e6:.0f} MB")
    assert used <= 1.25 * (3 * blocks + 4 * tables) + 100e6
    assert torch.equal(row_ptr, rp) and torch.equal(col_idx, ci) and torch.equal(val, 0.5 * va)
    assert sums == (nb * 32 * 0.0625, nb * 32 * 0.25, nb * 32 * 0.0625)
