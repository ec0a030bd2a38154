"""bs_spmm by the kernels that walk K in stages (csrc/bs_spmm_stream_kernel.h), at the sizes where they can
go wrong, against float64 and against the oracle."""
import pathlib
import subprocess
import sys

import numpy as np
import pytest
import torch

from oracle import bs_ref
from paper_1811_00206_amd import binding as bs

pytestmark = pytest.mark.gpu


def _product(M, nb, bank, k, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn((M, nb * bank), generator=g, device="cuda")
    if dtype == "f16":
        W = W.half()
    wide = bank > 256
    v, i = (bs.bs_prune_pack_wide if wide else bs.bs_prune_pack)(W, bank, k)
    dense = torch.zeros((M, nb, bank), dtype=torch.float64)
    dense.scatter_(2, i.cpu().to(torch.int64), v.cpu().double())
    return v, i, dense.view(M, nb * bank), g, bs.bs_spmm_wide if wide else bs.bs_spmm


def _check(Y, dense, x, terms):
    # a sum of n terms in fp32, in any order: off by at most n * 2^-24 of the sum of the terms'
    # magnitudes, and one more rounding per term
    bound = (terms + 1) * 2.0 ** -24 * (dense.abs() @ x.abs())
    assert ((Y.cpu().double() - dense @ x).abs() <= bound).all()


# every k the kernels are compiled for and two above; 0 to 3 banks beyond whole groups of four; one or several stages,
# slabs, wavefronts per workgroup and groups of them along K; 1 to 16 columns in the last tile
SHAPES = [
    # M, banks, bank, k, N, dtype
    (5, 17, 20, 4, 61, "f32"), (5, 41, 20, 4, 15, "f16"), (5, 18, 16, 5, 60, "f32"), (5, 11, 20, 6, 64, "f16"),
    (5, 9, 16, 7, 127, "f32"), (5, 15, 16, 8, 91, "f32"), (5, 7, 20, 9, 73, "f16"), (5, 12, 25, 10, 89, "f32"),
    (5, 5, 16, 11, 14, "f16"), (5, 10, 20, 12, 125, "f32"), (5, 13, 20, 13, 31, "f16"), (5, 15, 20, 14, 63, "f32"),
    (17, 6, 16, 15, 32, "f16"), (5, 33, 16, 16, 117, "f32"), (5, 8, 20, 17, 113, "f32"), (5, 7, 20, 20, 140, "f16"),
    (5, 68, 20, 5, 46, "f32"), (5, 67, 20, 20, 58, "f32"), (5, 26, 50, 11, 107, "f32"), (5, 25, 50, 20, 128, "f32"),
    (400, 51, 64, 33, 114, "f16"), (1000, 37, 64, 5, 60, "f32"), (5, 49, 16, 7, 62, "f32"), (5, 30, 100, 9, 94, "f32"),
    (700, 63, 50, 10, 115, "f32"), (1000, 25, 128, 17, 134, "f32"), (1000, 66, 64, 33, 139, "f32"), (200, 23, 256, 33, 132, "f32"),
    (300, 200, 64, 6, 16, "f16"),     # six slabs of one tile
]


@pytest.mark.parametrize("M,nb,bank,k,N,dtype", SHAPES)
def test_stages_against_float64(M, nb, bank, k, N, dtype):
    code = bs.BS_F16 if dtype == "f16" else bs.BS_F32
    assert bs.bs_spmm_plan(code, M, nb * bank, bank, k, N)["stages"] == 1
    v, i, dense, g, spmm = _product(M, nb, bank, k, dtype, M + nb + k)
    for pitch, start in ((N, 0), (N + 4 - N % 4, 0), (N + 9, 4)):
        print("stages", M, nb, bank, k, N, dtype, pitch, flush=True)
        X = torch.randn((nb * bank, pitch), generator=g, device="cuda")[:, start:start + N]
        if X.data_ptr() % 16:
            continue
        out = torch.full((M, N + 5), 7.0, device="cuda")
        Y = spmm(v, i, bank, X)
        _check(Y, dense, X.cpu().double(), nb * k)
        spmm(v, i, bank, X, out=out[:, :N])          # rows of Y further apart: nothing is written between them
        assert torch.equal(out[:, :N], Y) and bool((out[:, N:] == 7.0).all())


# launches that the second fit chooses: numbers of slabs that steps of a half would pass over, stages shorter than LDS allows
@pytest.mark.parametrize("M,nb,bank,k,N,dtype", [
    (16, 240, 20, 7, 31, "f16"), (17, 225, 32, 4, 46, "f32"), (16, 373, 25, 8, 58, "f32"), (16, 508, 25, 7, 32, "f16"),
    (95, 136, 32, 8, 181, "f32"), (145, 125, 64, 5, 37, "f16"), (78, 124, 64, 8, 502, "f32"), (512, 72, 64, 16, 196, "f32"),
    (165, 92, 32, 10, 235, "f16"), (233, 198, 25, 10, 234, "f16"), (1787, 97, 50, 17, 25, "f32")])
def test_launches_of_several_slabs(M, nb, bank, k, N, dtype):
    p = bs.bs_spmm_plan(bs.BS_F16 if dtype == "f16" else bs.BS_F32, M, nb * bank, bank, k, N)
    assert p["stages"] == 1 and p["stage_slabs"] > 1
    v, i, dense, g, spmm = _product(M, nb, bank, k, dtype, M + nb + k)
    X = torch.randn((nb * bank, N), generator=g, device="cuda")
    _check(spmm(v, i, bank, X), dense, X.cpu().double(), nb * k)


# 522 304 columns: four banks of X span more than 2 GB
@pytest.mark.parametrize("M,nb,bank,k,N,pitches", [
    (700, 63, 50, 10, 112, (113, 116, 121)), (700, 63, 50, 10, 115, (116, 117, 120)), (512, 72, 64, 16, 784, (785, 788)),
    (4000, 4, 256, 64, 100, (101, 104, 522304))])
def test_a_product_has_the_same_bits_for_every_row_pitch(M, nb, bank, k, N, pitches):
    assert bs.bs_spmm_plan(bs.BS_F32, M, nb * bank, bank, k, N)["stages"] == 1
    v, i, dense, g, spmm = _product(M, nb, bank, k, "f32", 7)
    X = torch.randn((nb * bank, N), generator=g, device="cuda")
    Y = spmm(v, i, bank, X)
    _check(Y, dense, X.cpu().double(), nb * k)
    for pitch in pitches:
        print("pitch", M, nb, bank, k, N, pitch, flush=True)
        wide = torch.empty((nb * bank, pitch), device="cuda")[:, :N]
        wide.copy_(X)
        out = torch.empty((M, N + 3), device="cuda")[:, :N]
        assert torch.equal(spmm(v, i, bank, wide, out=out), Y)


# both kernels of either type (k below 8, and from there on) with one stage, several in one half of LDS and several in two;
# 640: a group of four banks fills LDS
WIDE_SHAPES = [
    (5, 3, 264, 17, 64, "f32"), (5, 5, 264, 17, 15, "f16"), (5, 7, 264, 5, 15, "f32"), (5, 7, 264, 7, 15, "f16"),
    (5, 14, 400, 9, 1497, "f32"), (5, 14, 400, 8, 1497, "f16"), (5, 14, 400, 7, 1497, "f32"), (5, 14, 400, 6, 1497, "f16"),
    (5, 31, 264, 33, 1000, "f32"), (5, 18, 264, 9, 1497, "f16"), (5, 31, 300, 5, 1000, "f32"), (5, 37, 264, 6, 1000, "f16"),
    (5, 23, 512, 17, 15, "f16"), (100, 7, 640, 4, 1000, "f32"), (100, 7, 640, 4, 1000, "f16"), (351, 7, 512, 108, 1497, "f16"),
]


def test_the_16_bit_shapes_reach_every_kernel():
    seen = set()
    for M, nb, bank, k, N, dtype in WIDE_SHAPES:
        p = bs.bs_spmm_plan_wide(bs.BS_F16 if dtype == "f16" else bs.BS_F32, M, nb * bank, bank, k, N)
        assert p["stages"] == 1, (M, nb, bank, k, N, dtype)
        seen.add((dtype, k < 8, min(p["stage_slab_banks"], nb) > p["stage_banks"], p["stage_bufs"]))
    assert seen == {(d, few, s, b) for d in ("f32", "f16") for few in (True, False) for s, b in ((0, 1), (1, 1), (1, 2))}


@pytest.mark.parametrize("M,nb,bank,k,N,dtype", WIDE_SHAPES)
def test_16_bit_offsets_in_stages(M, nb, bank, k, N, dtype):
    v, i, dense, g, spmm = _product(M, nb, bank, k, dtype, bank + k)
    for pitch in (N, N + 4 - N % 4):
        print("16-bit offsets in stages", M, nb, bank, k, N, dtype, pitch, flush=True)
        X = torch.randn((nb * bank, pitch), generator=g, device="cuda")[:, :N]
        _check(spmm(v, i, bank, X), dense, X.cpu().double(), nb * k)


@pytest.mark.parametrize("bank,k,nb", [(512, 4, 9), (512, 7, 9), (600, 40, 6), (264, 9, 23)])
@pytest.mark.parametrize("M,N", [(300, 200), (1000, 37)])
def test_16_bit_offsets(bank, k, nb, M, N):
    """Products of the same kind that stay on the tile kernels."""
    assert bs.bs_spmm_plan_wide(bs.BS_F32, M, nb * bank, bank, k, N)["stages"] == 0
    print("16-bit offsets", bank, k, nb, M, N, flush=True)
    for dtype in ("f32", "f16"):
        v, i, dense, g, spmm = _product(M, nb, bank, k, dtype, bank + k)
        X = torch.randn((nb * bank, N), generator=g, device="cuda")
        _check(spmm(v, i, bank, X), dense, X.cpu().double(), nb * k)


def test_against_the_oracle_with_ties_and_zeros():
    M, nb, bank, k, N = 700, 63, 50, 10, 115
    rng = np.random.default_rng(3)
    W = rng.choice(np.array([-2.0, -1.0, 0.0, 0.5, 1.0, 2.0], dtype=np.float32), size=(M, nb * bank))
    X = rng.integers(-8, 9, size=(nb * bank, N)).astype(np.float32)
    v, i = bs.bs_prune_pack(torch.from_numpy(W).cuda(), bank, k)
    v_ref, i_ref = bs_ref.prune_pack(W, bank, k)
    # small integers and halves: every partial sum is exact, in any order
    assert np.array_equal(bs.bs_spmm(v, i, bank, torch.from_numpy(X).cuda()).cpu().numpy(), bs_ref.spmm(v_ref, i_ref, bank, X))


@pytest.mark.parametrize("N", [112, 115])
def test_infinities_stay_in_their_own_entries(N):
    """A row of X that no kept weight of a row of W refers to does not reach that row's result."""
    M, nb, bank, k = 700, 63, 50, 10
    v, i, dense, g, spmm = _product(M, nb, bank, k, "f32", 5)
    x = torch.randn((nb * bank, N), generator=g, device="cuda")
    x[nb * bank - 1] = float("inf")
    x[7] = float("nan")
    Y = spmm(v, i, bank, x).cpu()
    used = (dense[:, nb * bank - 1] != 0) | (dense[:, 7] != 0)
    assert 0 < int(used.sum()) < M
    assert bool(torch.isfinite(Y[~used]).all()) and not bool(torch.isfinite(Y[used]).any())


def test_a_capture_replays_what_the_eager_call_gives():
    M, nb, bank, k, N = 400, 51, 64, 33, 114
    v, i, dense, g, spmm = _product(M, nb, bank, k, "f32", 6)
    X = torch.randn((nb * bank, N), generator=g, device="cuda")
    eager = spmm(v, i, bank, X)
    Y = torch.empty_like(eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        spmm(v, i, bank, X, out=Y)
    for seed in range(3):
        X.normal_(generator=g)
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, spmm(v, i, bank, X))


# (M, K, bank, k, N): in stages
STAGED = (400, 3264, 64, 33, 114)           # the tile kernel of this shape needs its LDS limit raised
SMALL_TILE = (14019, 350, 50, 11, 36)       # ... and of this one not


@pytest.mark.parametrize("first,captured,refused", [
    (None, STAGED, True),                   # nothing has run: as bs.h says of a first use
    (None, SMALL_TILE, False),              # nothing needs preparing
    ((400, 656, 16, 3, 100), STAGED, False),    # the tile kernel of the captured shape has run, no stage kernel has
    ((6000, 3000, 100, 10, 128), STAGED, True),  # another stage kernel has run, and another tile kernel's shape
])
def test_which_kernel_a_capture_records_does_not_depend_on_what_has_run(first, captured, refused):
    """In a fresh process: a capture is refused, or records the kernel that the eager call launches."""
    code = f"""
import torch
from paper_1811_00206_amd import binding as bs
def product(M, K, bank, k, N):
    W = torch.randn((M, K), device="cuda")
    return *bs.bs_prune_pack(W, bank, k), bank, torch.randn((K, N), device="cuda")
captured, first = {captured}, {first}
torch.manual_seed(1)
p = bs.bs_spmm_plan(bs.BS_F32, *captured)
assert p["stages"] == 1 and (p["lds_bytes"] > 48 * 1024) == (captured == {STAGED})
if first:
    q = bs.bs_spmm_plan(bs.BS_F32, *first)
    assert q["lds_bytes"] > 48 * 1024
    assert {refused} or (q["stages"] == 0 and all(p[f] == q[f] for f in ("rows_kernel", "ch")))
    bs.bs_spmm(*product(*first))
args = product(*captured)
Y = torch.full((captured[0], captured[4]), 7.0, device="cuda")
torch.cuda.synchronize()
g, status = torch.cuda.CUDAGraph(), 0
with torch.cuda.graph(g):
    Y.mul_(1.0)
    try:
        bs.bs_spmm(*args, out=Y)
    except bs.BsError as e:
        status = e.status
for _ in range(3):
    g.replay()
    torch.cuda.synchronize()
    Z = bs.bs_spmm(*args) if not {refused} else torch.full_like(Y, 7.0)
    assert torch.equal(Y, Z)
    if not {refused}:
        Y.zero_()
        args[3].normal_()
print("RESULT", status)
"""
    print("captured", first, captured, flush=True)
    out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100,
                         cwd=str(pathlib.Path(__file__).resolve().parent.parent))
    assert out.returncode == 0 and f"RESULT {7 if refused else 0}\n" in out.stdout, out.stdout + out.stderr[-2000:]
