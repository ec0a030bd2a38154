"""The launches of the SpMM kernels that walk K in stages, checked on the host: every bank of X copied once to where
it is read, every bank walked once, the same barriers in every wavefront, LDS within a compute unit's; and the
generated code of every instantiation."""
import ctypes
import math
import os
import random
import re
import subprocess
import tempfile
import time
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_1811_00206_amd import binding as bs
from paper_1811_00206_amd import build as bs_build

P = 4                        # pieces of 4 columns per tile
BANKS = 16 // P              # banks side by side in LDS


def _copied(p, bank, banks, ragged):
    """LDS byte -> (row of X, piece) of one stage, as the copying wavefronts write it."""
    groups = -(-banks // BANKS)
    spare, quads, wrote = groups * BANKS - banks, (bank + 3) // 4, {}
    for wave in range(p["stage_copy_waves"]):
        g, rq = divmod(wave, quads)
        while g < groups:
            for lane in range(64):
                b, c, lrow = (lane & 15) // P, lane & (P - 1), lane >> 4
                last = 0 if b >= BANKS - spare else bank - 1 if ragged and b == BANKS - spare - 1 else bank
                if rq * 4 + lrow < (last if g == groups - 1 else bank):
                    at = (g * bank + rq * 4) * 256 + lane * 16
                    assert at not in wrote and at + 16 <= p["stage_buf_bytes"]
                    wrote[at] = ((g * BANKS + b) * bank + rq * 4 + lrow, c)
            g, rq = g + (rq + p["stage_copy_waves"]) // quads, (rq + p["stage_copy_waves"]) % quads
    return wrote


def _check(p, M, nb, bank, k, N, copies):
    where = str((M, nb, bank, k, N, p))
    slab, sb, ks, rows = p["stage_slab_banks"], p["stage_banks"], p["stage_ksplit"], p["stage_rows_per_wg"]
    assert p["stage_tiles"] * 4 * P >= N > (p["stage_tiles"] - 1) * 4 * P, where
    assert p["stage_slabs"] * slab >= nb > (p["stage_slabs"] - 1) * slab and p["stage_slabs"] <= p["n_slabs"], where
    assert p["stage_row_groups"] * rows >= M > (p["stage_row_groups"] - 1) * rows and rows <= 4 * P * p["stage_row_waves"], where
    assert sb % BANKS == 0 and slab % BANKS == 0 and p["stage_buf_bytes"] == sb * bank * 16 * P, where
    assert p["stage_bufs"] * p["stage_buf_bytes"] <= p["stage_lds_bytes"] <= 160 * 1024, where
    assert (ks - 1) * p["stage_row_waves"] * 1024 <= p["stage_lds_bytes"], where
    assert p["stage_copy_waves"] >= 1 and ks * p["stage_row_waves"] + p["stage_copy_waves"] <= 16, where
    for s in {0, p["stage_slabs"] - 1}:
        banks = min(slab, nb - s * slab)
        stages, groups, sg = -(-banks // sb), -(-banks // BANKS), sb // BANKS
        assert stages == 1 or sg % ks == 0, where
        barriers = stages + (stages - 1 if p["stage_bufs"] == 1 else 0)     # of a wavefront that copies
        walked = []
        for kq in range(ks):
            g, stage, first, end, met = kq, 0, 0, sg if stages > 1 else groups, 1
            while g < groups:
                if g >= end:
                    stage, met, first, end = stage + 1, met + 1 + (p["stage_bufs"] == 1), end, min(end + sg, groups)
                assert first <= g < end and (g - first + 1) * bank * 256 <= p["stage_buf_bytes"], where
                walked.append(g)
                g += ks
            assert met + (stages - 1 - stage) * (1 + (p["stage_bufs"] == 1)) == barriers, where
        assert sorted(walked) == list(range(groups)), where
        if copies:
            for stage, ragged in {(0, 0), (stages - 1, 1)}:
                sbk = min(sb, banks - stage * sb)
                wrote = _copied(p, bank, sbk, ragged)
                assert len(wrote) == (sbk * bank - ragged) * P, where
                for (at, (row, c)) in wrote.items():
                    j, r = divmod(row, bank)
                    assert at == ((j // BANKS) * bank + r) * 256 + (j % BANKS) * 16 * P + c * 16, where


def test_launches_of_random_shapes():
    rng = random.Random(811)
    taken = 0
    for n in range(3000):
        bank = rng.choice([4, 5, 8, 16, 25, 32, 50, 64, 100, 128, 255, 256])
        nb = rng.choice([1, 2, 3, 5, 7, 16, 30, 41, 60, 392])
        k = min(bank, rng.choice([*range(1, 18), 20, 32, 33, 63, 64, 128]))
        M = rng.choice([1, 3, 8, 37, 94, 128, 500, 1111, 6000, 16384])
        N = rng.choice([1, 8, 9, 13, 16, 17, 31, 32, 33, 37, 48, 49, 64, 100, 128, 784, 5000])
        dtype = rng.choice([bs.BS_F32, bs.BS_F16])
        try:
            p = bs.bs_spmm_plan(dtype, M, nb * bank, bank, k, N)
        except bs.BsError:
            continue
        assert p["stages"] in (0, 1)
        if p["stages"]:
            assert N > 8 and k >= 4
            taken += 1
            _check(p, M, nb, bank, k, N, bank * min(p["stage_banks"], nb) < 2000 and n % 3 == 0)
    assert taken > 500


def test_launches_of_random_shapes_with_16_bit_offsets():
    rng = random.Random(1811)
    taken = 0
    for n in range(3000):
        dtype = rng.choice([bs.BS_F32, bs.BS_F16])
        bank = rng.choice([264, 320, 400, 512, 600, 640, 648, 1024])
        nb = rng.choice([1, 2, 3, 5, 7, 9, 14, 18, 31, 37])
        k = rng.choice([*range(1, 18), 20, 33, 64, 128])
        M = rng.choice([1, 5, 37, 94, 351, 1111, 6000, 16384])
        N = rng.choice([8, 9, 15, 33, 64, 100, 784, 1000, 1497])
        try:
            p = bs.bs_spmm_plan_wide(dtype, M, nb * bank, bank, k, N)
        except bs.BsError:
            continue
        if p["stages"]:
            assert N > 8 and k >= 4 and bank <= 640     # four banks of 640 fill LDS
            taken += 1
            _check(p, M, nb, bank, k, N, n % 12 == 0)
    assert taken > 150


@pytest.mark.parametrize("dtype,shape,stages,slabs", [
    (bs.BS_F16, (1963, 23552, 512, 25, 13), 0, 12), (bs.BS_F32, (291, 20400, 300, 45, 172), 1, 9)])
def test_products_with_16_bit_offsets_keep_their_launches(dtype, shape, stages, slabs):
    """The expected times of these are a fit to launches whose slabs were looked for in steps of a half."""
    p = bs.bs_spmm_plan_wide(dtype, *shape)
    assert (p["stages"], p["stage_slabs"] if stages else p["n_slabs"]) == (stages, slabs)


def test_the_timed_sizes_and_small_ones():
    for M, K, bank, k, N, dtype in [(6000, 3000, 100, 10, 128, bs.BS_F32), (6000, 3000, 50, 15, 37, bs.BS_F32),
                                    (512, 4608, 64, 16, 784, bs.BS_F32), (4096, 25088, 64, 6, 16, bs.BS_F16),
                                    (512, 6400, 64, 16, 5000, bs.BS_F32)]:
        p = bs.bs_spmm_plan(dtype, M, K, bank, k, N)
        assert p["stages"] == 1
        _check(p, M, K // bank, bank, k, N, True)
    assert bs.bs_spmm_plan(bs.BS_F32, 6000, 3000, 100, 10, 8)["stages"] == 0        # few columns: the chunk walk
    assert bs.bs_spmm_plan(bs.BS_F32, 256, 256, 64, 16, 32)["stages"] == 0          # a few microseconds
    assert bs.bs_spmm_plan(bs.BS_F32, 6000, 3000, 100, 3, 128)["stages"] == 0       # fewer than four per bank
    # one tile of columns and more than 32 entries per bank; an X of more than 128 MB
    assert bs.bs_spmm_plan(bs.BS_F32, 700, 6144, 128, 33, 16)["stages"] == 0
    assert bs.bs_spmm_plan(bs.BS_F32, 512, 6400, 64, 16, 5001)["stages"] == 0


@pytest.mark.parametrize("dtype,M,K,bank,k,N", [
    (bs.BS_F16, 4096, 25088, 64, 6, 16), (bs.BS_F32, 879, 12400, 100, 8, 20), (bs.BS_F16, 108, 19125, 25, 10, 251)])
def test_planning_many_slabs_costs_little(dtype, M, K, bank, k, N):
    """Every call plans its launch.  A host query of this product against one of 8 columns, which only the tile kernels'
    planning is needed for: 3.1 to 4.3 times as long if every launch is priced in full, 1.5 to 2.0 as it is."""
    plan, out, best = bs.load_library().bs_spmm_plan, (ctypes.c_int64 * 30)(), {N: math.inf, 8: math.inf}
    for _ in range(300):             # in turn and in pieces of some 100 us: what else the host does meets both alike
        for n in best:
            t = time.perf_counter()
            for _ in range(60):
                plan(dtype, M, K, bank, k, n, out, 30)
            best[n] = min(best[n], time.perf_counter() - t)
    assert best[N] < 2.7 * best[8]


def _chain(parts):
    """The parts (last axis: exact products or sums in fp32) added one after the other, each addition rounded to fp32."""
    total = np.zeros(parts.shape[:-1], np.float32)
    for i in range(parts.shape[-1]):
        total = (total.astype(np.float64) + parts[..., i]).astype(np.float32)
    return total


def _tile_sums(p, t):
    """The tile kernels' order: [sums, banks, k] products -> fp32 sums."""
    slabs = []
    for s in range(p["n_slabs"]):
        run = t[:, s * p["sb"]:(s + 1) * p["sb"]].reshape(len(t), -1)
        chunks = run.reshape(len(t), -1, p["ch"])
        lanes = [_chain(chunks[:, lane::p["lpr"]].reshape(len(t), -1)) for lane in range(p["lpr"])]
        while len(lanes) > 1:       # the exchange between lanes
            lanes = [lanes[i] + lanes[i + 1] for i in range(0, len(lanes), 2)]
        slabs.append(lanes[0])
    return _chain(np.stack(slabs, -1))


def _stage_sums(p, t):
    """The stage kernels' order."""
    nb, k, slabs = t.shape[1], t.shape[2], []
    sg, ks = p["stage_banks"] // BANKS, p["stage_ksplit"]
    for s in range(p["stage_slabs"]):
        banks = t[:, s * p["stage_slab_banks"]:(s + 1) * p["stage_slab_banks"]]
        groups = -(-banks.shape[1] // BANKS)
        banks = np.pad(banks, [(0, 0), (0, groups * BANKS - banks.shape[1]), (0, 0)]).reshape(len(t), groups, BANKS, k)
        waves = []
        for kq in range(ks):
            stages = []
            for first in range(0, groups, sg):
                mine = banks[:, first:first + sg][:, kq::ks] if groups > sg else banks[:, kq::ks]
                stages.append(_chain(mine.transpose(0, 2, 1, 3).reshape(len(t), BANKS, -1)))
            lane = _chain(np.stack(stages, -1))
            waves.append((lane[:, 0] + lane[:, 1]) + (lane[:, 2] + lane[:, 3]))
        slabs.append(_chain(np.stack(waves, -1)))
    return _chain(np.stack(slabs, -1))


def test_products_whose_sums_would_round_worse_stay_on_the_tile_kernels():
    # odd row lengths and small tiles, which the tile kernels walk with up to 64 lanes per row
    for shape in [(6722, 144, 16, 13, 40), (3700, 350, 50, 25, 17), (146, 384, 128, 43, 1375), (6109, 300, 100, 38, 53),
                  (14391, 384, 128, 31, 9), (2387, 500, 100, 33, 32), (3432, 400, 100, 45, 43)]:
        p = bs.bs_spmm_plan(bs.BS_F32, *shape)
        assert p["stages"] == 0 and p["lpr"] >= 8, (shape, p)


@pytest.mark.parametrize("dtype,shape", [
    (bs.BS_F32, (3833, 5120, 256, 95, 30)), (bs.BS_F32, (2565, 14208, 128, 42, 21)), (bs.BS_F16, (520, 400, 100, 5, 5799)),
    (bs.BS_F32, (861, 1800, 50, 4, 17))])
def test_products_that_are_slower_in_stages_stay_on_the_tile_kernels(dtype, shape):
    """Long banks with a large stream of W, and tiles of few columns: 27.4, 43.4, 21.0 and 6.5 us by tiles, 42.7, 62.8, 30.2 and 8.5
    in stages."""
    assert bs.bs_spmm_plan(dtype, *shape)["stages"] == 0


# shape, and the launch that the first fit gives it: slabs, banks per slab and per stage, wavefronts along K
@pytest.mark.parametrize("dtype,shape,first", [
    (bs.BS_F32, (512, 4608, 64, 16, 784), (1, 72, 16, 2)), (bs.BS_F32, (512, 4608, 64, 16, 196), (1, 72, 12, 3)), (bs.BS_F32, (64, 10880, 128, 28, 2441), (3, 32, 8, 2)),
    (bs.BS_F32, (188, 13200, 100, 6, 12), (6, 24, 24, 6)), (bs.BS_F16, (472, 21792, 32, 14, 96), (4, 172, 32, 4)),
    (bs.BS_F32, (2900, 3648, 64, 31, 73), (1, 60, 12, 3)), (bs.BS_F32, (6000, 3000, 50, 15, 37), (1, 60, 24, 1))])
def test_a_faster_launch_rounds_no_worse(dtype, shape, first):
    """What the second fit expects to be faster is taken only where its sums are no less exact: both orders of addition on
    the same products, against 64 bits."""
    p = bs.bs_spmm_plan(dtype, *shape)
    assert p["stages"] == 1
    _, K, bank, k, _ = shape
    g = np.random.default_rng(K + k)
    n = 40000 * 64 // (K // bank * k)
    w, x = (g.standard_normal((n, K // bank, k)).astype(np.float32) for _ in range(2))
    t = w.astype(np.float64) * x
    exact = t.sum(axis=(1, 2))
    before = dict(zip(("stage_slabs", "stage_slab_banks", "stage_banks", "stage_ksplit"), first))
    was, now = (np.linalg.norm(_stage_sums(q, t) - exact) for q in (before, p))
    # each norm is over n independent errors: known to about 1 / sqrt(2 n) of itself
    assert now <= was * (1 + 3 / math.sqrt(n)), (p, now / was)


# the first five close to the line; many banks; the timed sizes
@pytest.mark.parametrize("M,K,bank,k,N", [
    (6774, 320, 64, 19, 54), (2880, 336, 16, 6, 81), (9038, 400, 100, 4, 29), (245, 550, 50, 5, 543), (1591, 768, 64, 13, 15),
    (700, 3150, 50, 10, 115), (400, 3264, 64, 33, 114), (6000, 3000, 100, 10, 128), (6000, 3000, 50, 15, 37), (512, 4608, 64, 16, 784)])
def test_sums_are_no_less_exact_than_the_tile_kernels(M, K, bank, k, N):
    """Both orders of addition on the same products, against 64 bits."""
    p = bs.bs_spmm_plan(bs.BS_F32, M, K, bank, k, N)
    assert p["stages"] == 1
    g = np.random.default_rng(K + k)
    n = 40000 * 64 // (K // bank * k)
    w, x = (g.standard_normal((n, K // bank, k)).astype(np.float32) for _ in range(2))
    t = w.astype(np.float64) * x
    exact = t.sum(axis=(1, 2))
    tiles, stages = (np.linalg.norm(sums(p, t) - exact) for sums in (_tile_sums, _stage_sums))
    # each norm is over n independent errors: known to about 1 / sqrt(2 n) of itself
    assert stages <= tiles * (1 + 3 / math.sqrt(n)), (p, stages / tiles)


SOURCES = ["bs_spmm_stream_f32.hip", "bs_spmm_stream_f16.hip", "bs_spmm_stream_wide.hip"]


@pytest.fixture(scope="module")
def texts():
    def assembly(src):
        out = tempfile.NamedTemporaryFile(suffix=".s", delete=False).name
        flags = [f for f in bs_build.FLAGS if f != "-fPIC"]
        subprocess.check_call([bs_build.HIPCC, *flags, "-S", "--cuda-device-only", "-o", out, os.path.join(bs_build.CSRC, src)],
                              stderr=subprocess.DEVNULL)
        text = open(out).read()
        os.unlink(out)
        return text
    with ThreadPoolExecutor(3) as ex:
        return list(ex.map(assembly, SOURCES))


def test_generated_code(texts):
    """No scratch memory; between a direct-to-LDS copy and the next barrier there is a wait for every load (the
    compiler does not track these copies itself)."""
    kernels = 0
    for text in texts:
        assert all(int(n) == 0 for n in re.findall(r"\.vgpr_spill_count:\s+(\d+)", text))
        assert all(int(n) == 0 for n in re.findall(r"\.private_segment_fixed_size:\s+(\d+)", text))
        # 128 registers: 16 wavefronts on a compute unit
        assert all(int(n) <= 128 for n in re.findall(r"\.vgpr_count:\s+(\d+)", text))
        name, pending, copies = None, False, 0
        for line in text.splitlines():
            s = line.strip()
            m = re.match(r"^(_ZN2bs18spmm_stream_kernel\w+):", line)
            if m:
                name, pending, copies = m.group(1), False, 0
            elif name is None:
                continue
            elif s.startswith(".Lfunc_end"):
                assert copies == 2, name         # the first stage's and the later ones'
                kernels, name = kernels + 1, None
            elif s.startswith("global_load_lds"):
                pending, copies = True, copies + 1
            elif s.startswith("s_waitcnt") and "vmcnt(0)" in s:
                pending = False
            elif s.startswith("s_barrier"):
                assert not pending, name
    assert kernels == 2 * 14 + 4
