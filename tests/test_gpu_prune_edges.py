"""bs_prune_pack / bs_prune_pack_wide where their lane layouts change: banks around every
multiple of what a lane owns, matrices whose last wavefront holds few banks, and keys that
agree down to the last bits.  vals/idx bit for bit against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import bs_ref
from paper_1811_00206_amd import binding as bs

pytestmark = pytest.mark.gpu


def _weights(kind, M, K, dtype, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    if kind == "gauss":
        W = rng.standard_normal((M, K), dtype=np.float32)
    elif kind == "ties":        # three magnitudes, random signs
        W = (rng.integers(0, 3, (M, K)) * rng.choice([-1.0, 1.0], (M, K))).astype(np.float32)
    else:                       # magnitudes that differ in the lowest bits of the type only
        step = 2.0 ** (-23 if dtype == "f32" else -10)
        W = ((1 + rng.integers(0, 200, (M, K)) * step) * rng.choice([-1.0, 1.0], (M, K))).astype(np.float32)
    return W if dtype == "f32" else W.astype(np.float16)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("bank", [1, 2, 15, 16, 17, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256,
                                  512, 520, 1024, 1032, 2048])
def test_prune_pack_layout_edges(bank, dtype):
    wide = bank > 256
    prune = bs.bs_prune_pack_wide if wide else bs.bs_prune_pack
    for kind in ("gauss", "ties", "low_bits"):
        for rows, nb in ((1, 1), (3, 3), (67, 2)):
            for k in sorted({1, (bank + 1) // 2, bank}):
                print("prune edges", bank, dtype, kind, rows, nb, k, flush=True)
                W = _weights(kind, rows, nb * bank, dtype, bank + k)
                v, i = prune(torch.from_numpy(W).to("cuda:0"), bank, k)
                v_ref, i_ref = bs_ref.prune_pack(W, bank, k, wide=wide)
                assert i.cpu().numpy().tobytes() == i_ref.tobytes(), (kind, rows, nb, k)
                assert v.cpu().numpy().tobytes() == v_ref.tobytes(), (kind, rows, nb, k)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("bank", [3, 4, 5])
def test_prune_pack_smallest_banks(bank, dtype):
    """Around the four elements up to which fp32 lanes have a kernel of their own; four, the
    smallest whole piece, with 16-bit offsets too."""
    test_prune_pack_layout_edges(bank, dtype)
    if bank == 4 and dtype == "f32":
        for kind in ("gauss", "ties", "low_bits"):
            for k in (1, 2, 4):
                W = _weights(kind, 67, 5 * bank, dtype, k)
                v, i = bs.bs_prune_pack_wide(torch.from_numpy(W).to("cuda:0"), bank, k)
                v_ref, i_ref = bs_ref.prune_pack(W, bank, k, wide=True)
                assert i.cpu().numpy().tobytes() == i_ref.tobytes() and v.cpu().numpy().tobytes() == v_ref.tobytes()


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("k", [1, 3, 4, 5, 16, 32, 33, 64, 100, 128, 129, 131, 255, 256])
def test_reprune_edges(k, dtype):
    """bs_reprune where the way to the stored offsets changes: survivors of a wavefront around one
    and four per lane, stored offsets in whole 16-byte pieces or not, last groups that end inside
    a piece."""
    lanes = next(n for n in (1, 2, 4, 8) if k <= 32 * n)
    per_wave = 64 // lanes
    bank = min(256, 2 * k)
    kept = {1, 2, 64 // per_wave, 64 // per_wave + 1, 256 // per_wave, 256 // per_wave + 1, k - 1, k}
    for rows, nb in ((1, 1), (3, 3), (67, 2)):
        v, i = bs_ref.prune_pack(_weights("ties" if rows == 3 else "gauss", rows, nb * bank, dtype, k), bank, k)
        vd, idd = torch.from_numpy(v).to("cuda:0"), torch.from_numpy(i).to("cuda:0")
        for k2 in sorted(n for n in kept if 1 <= n <= k):
            print("reprune edges", k, dtype, rows, nb, k2, flush=True)
            v2, i2 = bs.bs_reprune(vd, idd, bank, k2)
            v_ref, i_ref = bs_ref.reprune(v, i, k2)
            assert i2.cpu().numpy().tobytes() == i_ref.tobytes(), (rows, nb, k2)
            assert v2.cpu().numpy().tobytes() == v_ref.tobytes(), (rows, nb, k2)
