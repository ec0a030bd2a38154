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


@pytest.mark.parametrize("first,captured", [(4, 2), (2, 4)])
def test_a_first_product_prepares_the_capture_of_another_width(first, captured):
    """One to three columns run in a kernel of their own.  A product outside a capture prepares
    both kernels of its shape, as it did when there was one.  Run in a fresh process."""
    import pathlib
    import subprocess
    import sys
    code = f"""
import torch
from paper_1811_00206_amd import binding as bs
W = torch.randn((300, 4096), device="cuda")
v, i = bs.bs_prune_pack(W, 64, 6)
X = {{n: torch.randn((4096, n), device="cuda") for n in (2, 4)}}
p = {{n: bs.bs_spmm_plan(bs.BS_F32, 300, 4096, 64, 6, n) for n in (2, 4)}}
assert p[2]["lds_bytes"] > 48 * 1024 and all(p[2][f] == p[4][f] for f in ("ch", "lpr", "u", "rows_kernel"))
bs.bs_spmm(v, i, 64, X[{first}])
torch.cuda.synchronize()
Y = torch.empty((300, {captured}), device="cuda")
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g):
    bs.bs_spmm(v, i, 64, X[{captured}], out=Y)
Y.zero_()
g.replay()
torch.cuda.synchronize()
assert torch.equal(Y, bs.bs_spmm(v, i, 64, X[{captured}]))
print("RESULT captured")
"""
    print("capture after another width", first, captured, flush=True)
    out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100,
                         cwd=str(pathlib.Path(__file__).resolve().parent.parent))
    assert out.returncode == 0 and "RESULT captured" in out.stdout, out.stdout + out.stderr[-2000:]
