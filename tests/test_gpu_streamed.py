"""bs_spmv on packed matrices that are larger than the last-level cache (spmv_streamed_kernel, csrc/bs_spmv_kernel.h): every
chunk width and number of chunk slots, and those of them that keep the ordinary loads, against float64 on rows from everywhere."""
import pytest
import torch

from paper_1811_00206_amd import binding as bs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BYTES = 256 << 20

# chunks of 4, 2 and 1 (fp32), 8, 4, 2 and 1 (binary16) entries; one round of 5 to 8 slots, several rounds; 16-bit offsets
SHAPES = [
    # banks, bank, k, dtype
    (33, 64, 40, "f32"), (31, 100, 50, "f32"), (77, 50, 19, "f32"), (64, 256, 128, "f32"), (97, 128, 64, "f16"), (83, 100, 50, "f16"),
    (99, 100, 52, "f16"), (97, 64, 33, "f16"), (40, 50, 30, "f32"), (40, 64, 40, "f32"), (16, 1024, 200, "f32"), (15, 512, 201, "f32"), (32, 512, 100, "f16"),
]


# short rows (8 to 32 lanes) and an x that does not fit LDS, which have no kernels with such loads
OTHERS = [(64, 64, 16, "f16"), (32, 128, 16, "f32"), (16, 64, 16, "f16"), (4, 64, 8, "f32"), (161, 256, 13, "f32"), (20, 512, 16, "f32")]


@pytest.mark.parametrize("nb,bank,k,dtype", SHAPES)
def test_matrices_larger_than_the_last_level_cache(nb, bank, k, dtype):
    _check(nb, bank, k, dtype, True)


@pytest.mark.parametrize("nb,bank,k,dtype", OTHERS)
def test_large_matrices_without_kernels_of_their_own(nb, bank, k, dtype):
    _check(nb, bank, k, dtype, False)


def _check(nb, bank, k, dtype, streamed):
    wide = bank > 256
    vt, it = (torch.float16, torch.float32)[dtype == "f32"], (torch.uint8, torch.uint16)[wide]
    entry = (2 if dtype == "f16" else 4) + (2 if wide else 1)
    M = BYTES // (nb * k * entry) + 3
    assert M * nb * k * entry > BYTES
    print("streamed", M, nb, bank, k, dtype, flush=True)
    if not wide:
        p = bs.bs_spmv_plan(bs.BS_F16 if dtype == "f16" else bs.BS_F32, M, nb * bank, bank, k)
        assert streamed == (p["lpr"] == 64 and not p["slab_kernel"])
    g = torch.Generator(device="cuda").manual_seed(nb + k)
    vals = torch.empty((M, nb, k), dtype=vt, device=DEV)
    vals.view(-1)[:] = torch.randn(M * nb * k, generator=g, device=DEV, dtype=vt)
    idx = torch.randint(0, bank, (M, nb, k), generator=g, device=DEV, dtype=torch.int32).to(torch.int16).view(it) if wide else torch.randint(
        0, bank, (M, nb, k), generator=g, device=DEV, dtype=torch.uint8)
    x = torch.randn(nb * bank, generator=g, device=DEV)
    y = (bs.bs_spmv_wide if wide else bs.bs_spmv)(vals, idx, bank, x)
    rows = torch.tensor([0, 1, 2, 3, M // 3, M // 2, M - 5, M - 4, M - 3, M - 2, M - 1], device=DEV)
    at = (idx.view(torch.int16) if wide else idx)[rows].long() + bank * torch.arange(nb, device=DEV)[None, :, None]
    terms = vals[rows].double() * x.double()[at]
    # n terms in fp32, in any order: off by at most n * 2^-24 of the sum of the terms' magnitudes
    bound = (nb * k + 1) * 2.0 ** -24 * terms.abs().sum((1, 2))
    assert ((y[rows].double() - terms.sum((1, 2))).abs() <= bound).all()


@pytest.mark.parametrize("nb,bank,k,dtype", [(33, 64, 5, "f32"), (41, 100, 9, "f32"), (16, 256, 30, "f32"), (77, 51, 6, "f16"), (64, 128, 8, "f16"),
                                             (16, 512, 16, "f32"), (9, 1024, 8, "f16")])
def test_pruning_of_matrices_larger_than_the_last_level_cache(nb, bank, k, dtype):
    """prune_pack_kernel's non-temporal copies: rows from everywhere against the same rows pruned by themselves."""
    size = 2 if dtype == "f16" else 4
    M = BYTES // (nb * bank * size) + 5
    assert M * nb * bank * size > BYTES
    print("streamed prune", M, nb, bank, k, dtype, flush=True)
    g = torch.Generator(device="cuda").manual_seed(nb + k)
    W = torch.randn((M, nb * bank), generator=g, device=DEV, dtype=torch.float16 if dtype == "f16" else torch.float32)
    prune = bs.bs_prune_pack_wide if bank > 256 else bs.bs_prune_pack
    vals, idx = prune(W, bank, k)
    view = lambda t: t.view(torch.int16) if t.dtype == torch.uint16 else t
    for first in (0, M // 3, M - 64):
        v, i = prune(W[first:first + 64].clone(), bank, k)
        assert torch.equal(vals[first:first + 64], v) and torch.equal(view(idx)[first:first + 64], view(i))
