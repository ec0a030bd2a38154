"""bs_spmm where the tile of X is brought in by more wavefronts than walk rows (few rows per
workgroup), and where rows of X start at any multiple of 4 bytes; against float64."""
import pytest
import torch

from paper_1811_00206_amd import binding as bs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bank,k", [(16, 3), (64, 16), (512, 40)])
@pytest.mark.parametrize("M", [1, 9, 200])
@pytest.mark.parametrize("N", [2, 5, 15, 17, 31, 32, 33, 37, 64, 101])
def test_copied_tiles(bank, k, M, N):
    print("copied tiles", bank, k, M, N, flush=True)
    K = 2048
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N)
    prune, spmm = (bs.bs_prune_pack_wide, bs.bs_spmm_wide) if bank > 256 else (bs.bs_prune_pack, bs.bs_spmm)
    W = torch.randn((M, K), generator=g, device="cuda")
    v, i = prune(W, bank, k)
    dense = torch.zeros((M, K // bank, bank), dtype=torch.float64)
    dense.scatter_(2, i.cpu().to(torch.int64), v.cpu().double())
    dense = dense.view(M, K)
    wide = torch.randn((K, N + 9), generator=g, device="cuda")
    for X in (wide[:, :N].contiguous(), wide[:, 4:4 + N] if (N + 9) % 4 == 0 else wide[:, :N]):
        Y = spmm(v, i, bank, X).cpu().double()
        x = X.cpu().double()
        # a sum of n = K/bank*k terms in fp32, in any order: off by at most n * 2^-24 of the
        # sum of the terms' magnitudes, and one more rounding per term
        bound = (K // bank * k + 1) * 2.0 ** -24 * (dense.abs() @ x.abs())
        assert ((Y - dense @ x).abs() <= bound).all()


@pytest.mark.parametrize("bank,k", [(16, 3), (25, 7), (512, 40)])
@pytest.mark.parametrize("M,nb", [(1, 1), (9, 5), (300, 17), (2100, 41)])
@pytest.mark.parametrize("N", [1, 2, 3, 5])
def test_few_columns(bank, k, M, nb, N):
    """The kinds of copy and the workgroup sizes meet here: one to three columns in rows that are
    adjacent or lie further apart, tiles of less than a wavefront's rows and of many times a
    workgroup's."""
    K = nb * bank
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + K + N)
    prune, spmm = (bs.bs_prune_pack_wide, bs.bs_spmm_wide) if bank > 256 else (bs.bs_prune_pack, bs.bs_spmm)
    W = torch.randn((M, K), generator=g, device="cuda")
    v, i = prune(W, bank, k)
    dense = torch.zeros((M, nb, bank), dtype=torch.float64)
    dense.scatter_(2, i.cpu().to(torch.int64), v.cpu().double())
    dense = dense.view(M, K)
    for pitch in (N, N + 1, 7):
        print("few columns", bank, k, M, nb, N, pitch, flush=True)
        X = torch.randn((K, pitch), generator=g, device="cuda")[:, :N]
        x = X.cpu().double()
        # as above
        bound = (nb * k + 1) * 2.0 ** -24 * (dense.abs() @ x.abs())
        assert ((spmm(v, i, bank, X).cpu().double() - dense @ x).abs() <= bound).all()
