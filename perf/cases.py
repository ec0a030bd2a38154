"""The work that a user of this library has it do, as cases that can be timed.

Each case is one call sequence through the Python names of the C ABI
(``paper_1811_00206_amd.binding``) on synthetic matrices: products with one
column (``spmv``) and with several (``spmm``), LSTM sequences, and the pruning
of a dense matrix (``prune``) or of a packed one (``reprune``) when a model is
loaded.  The sizes are those of ``paper_1811_00206_amd.workloads`` and generic
ones around them.

A case is a dict: ``op``; ``M``, ``K`` (rows and columns of the matrix; for
``lstm`` M = 4H gate rows and K = I + H columns), ``bank`` (balance range) and
``k`` (weights kept per bank), ``dtype`` of the stored weights; ``N`` columns of
X for ``spmm``, ``T`` steps for ``lstm``, ``k2`` for ``reprune``.  Banks over 256
use the entry points with 16-bit offsets.
"""
from __future__ import annotations

import math

import torch

from paper_1811_00206_amd import binding as bs

# no drawn case moves more bytes or does more multiply-adds than the largest listed ones
MAX_BYTES = 336_000_000
MAX_FLOPS = 925_000_000


def _case(op, M, K, bank, k, dtype="f32", **more):
    return {"op": op, "M": M, "K": K, "bank": bank, "k": k, "dtype": dtype, **more}


def listed():
    return [
        # the smallest call: a 256 x 256 matrix at 75 % sparsity (launch and call overhead)
        dict(name="spmv_256x256", **_case("spmv", 256, 256, 64, 16)),
        # one time step's gate product of a 1500-unit LSTM at 90 % sparsity
        dict(name="spmv_lstm1500", **_case("spmv", 6000, 3000, 100, 10)),
        # VGG-16 fc6 at batch 1, weights stored as binary16
        dict(name="spmv_fc6_f16", **_case("spmv", 4096, 25088, 64, 6, "f16")),
        # the largest product with a vector: the 16384 x 8192 benchmark matrix at 50 %
        dict(name="spmv_16k_half", **_case("spmv", 16384, 8192, 256, 128)),
        # the LSTM gate product for a small and for a large batch
        dict(name="spmm_lstm1500_n8", **_case("spmm", 6000, 3000, 100, 10, N=8)),
        dict(name="spmm_lstm1500_n128", **_case("spmm", 6000, 3000, 100, 10, N=128)),
        # a ragged batch (37 sequences left in a group) on Table 4's balance range of 50
        dict(name="spmm_ragged_n37", **_case("spmm", 6000, 3000, 50, 15, N=37)),
        # fc6 at batch 16, binary16 weights
        dict(name="spmm_fc6_f16_n16", **_case("spmm", 4096, 25088, 64, 6, "f16", N=16)),
        # a 512 x 512 x 3 x 3 convolution over a 28 x 28 output as an im2col product
        dict(name="spmm_conv_n784", **_case("spmm", 512, 4608, 64, 16, N=784)),
        # model load: pruning and packing a dense matrix in either storage type
        dict(name="prune_lstm1500", **_case("prune", 6000, 3000, 100, 10)),
        dict(name="prune_fc6_f16", **_case("prune", 4096, 25088, 64, 6, "f16")),
        # recurrent inference: 32 dependent steps of the 1500-unit LSTM
        dict(name="lstm1500_t32", **_case("lstm", 6000, 3000, 100, 10, T=32)),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case of the same ranges: the size of the matrix over four orders of
    magnitude, odd row and column counts, 50 to 97 % sparsity, balance ranges 16..1024
    (over 256: 16-bit offsets), both storage types."""
    while True:
        op = rng.choices(("spmv", "spmm", "prune", "lstm", "reprune"), (5, 7, 4, 3, 1))[0]
        dtype = rng.choice(("f32", "f32", "f16"))
        bank = rng.choice((16, 25, 32, 50, 64, 64, 100, 100, 128, 256, 512, 1024))
        k = max(1, round(bank * _log_uniform(rng, 0.03, 0.5)))
        if bank > 256 and op in ("lstm", "reprune"):
            continue
        if op == "lstm":
            H = 4 * round(_log_uniform(rng, 128, 1536) / 4)
            # input size: whatever makes [x ; h] a whole number of banks, a multiple of 4
            nb = math.ceil((H + _log_uniform(rng, 128, 1536)) / bank)
            while (nb * bank) % 4:
                nb += 1
            M, K = 4 * H, nb * bank
        else:
            M = round(_log_uniform(rng, 64, 16384))
            K = bank * max(1, round(_log_uniform(rng, 256, 25088) / bank))
        case = _case(op, M, K, bank, k, dtype)
        if op == "spmm":
            case["N"] = round(_log_uniform(rng, 2, 50176))
        elif op == "lstm":
            case["T"] = round(_log_uniform(rng, 1, 32))
        elif op == "reprune":
            case["k2"] = max(1, k // 2)
        w = work(case)
        if M * K <= 16384 * 8192 and w["bytes"] <= MAX_BYTES and w["flops"] <= MAX_FLOPS:
            return case


def _uniform(gen, *shape, a=1.0):
    return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-a, a, generator=gen)


def prepare(case, seed):
    """Weights ~ N(0, 1/sqrt(K)) (a trained layer's spread), activations ~ U(-1, 1); products
    start from the packed matrix, as a program that has loaded its model does."""
    op, M, K, bank, k = case["op"], case["M"], case["K"], case["bank"], case["k"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.float32) * (K ** -0.5)
    if case["dtype"] == "f16":
        W = W.half()
    state = {"op": op, "bank": bank, "wide": bank > 256}
    if op == "prune":
        state["W"], state["k"] = W, k
        return state
    prune = bs.bs_prune_pack_wide if bank > 256 else bs.bs_prune_pack
    state["vals"], state["idx"] = prune(W, bank, k)
    if op == "spmv":
        state["x"] = _uniform(gen, K)
    elif op == "spmm":
        state["X"] = _uniform(gen, K, case["N"])
    elif op == "reprune":
        state["k2"] = case["k2"]
    elif op == "lstm":
        H = M // 4
        state["X"] = _uniform(gen, case["T"], K - H)
        state["h0"], state["c0"] = _uniform(gen, H), _uniform(gen, H)
        state["bias"] = _uniform(gen, M, a=0.5)
    return state


def run(state):
    op, bank = state["op"], state["bank"]
    if op == "spmv":
        product = bs.bs_spmv_wide if state["wide"] else bs.bs_spmv
        return product(state["vals"], state["idx"], bank, state["x"])
    if op == "spmm":
        product = bs.bs_spmm_wide if state["wide"] else bs.bs_spmm
        return product(state["vals"], state["idx"], bank, state["X"])
    if op == "prune":
        prune = bs.bs_prune_pack_wide if state["wide"] else bs.bs_prune_pack
        return prune(state["W"], bank, state["k"])
    if op == "reprune":
        return bs.bs_reprune(state["vals"], state["idx"], bank, state["k2"])
    c = state["c0"].clone()     # the cell state is updated in place
    H_all = bs.bs_lstm_sequence(state["vals"], state["idx"], bank, state["X"], state["h0"],
                                state["bias"], c)
    return H_all, c


def work(case):
    op, M, K, bank, k = case["op"], case["M"], case["K"], case["bank"], case["k"]
    val = 4 if case["dtype"] == "f32" else 2
    off = 1 if bank <= 256 else 2
    nnz = M * (K // bank) * k
    packed = nnz * (val + off)
    if op == "prune":
        return {"bytes": M * K * val + packed, "flops": 0}
    if op == "reprune":
        return {"bytes": packed + M * (K // bank) * case["k2"] * (val + off), "flops": 0}
    if op == "lstm":
        T, H = case["T"], M // 4
        # weights, bias and states once; an input row and a hidden state per step
        return {"bytes": packed + 4 * (M + 3 * H) + 4 * T * (K - H) + 4 * T * H, "flops": 2 * nnz * T}
    N = case.get("N", 1)
    return {"bytes": packed + 4 * K * N + 4 * M * N, "flops": 2 * nnz * N}


def tolerance(case):
    """Compared with the same call in float64 (50 cases of these ranges): products differ by up
    to 4e-7 (2-norm) and 2.7e-6 (largest element, over the rms), sequences by 2.1e-7 and 9e-7;
    four times that is stated."""
    if case["op"] in ("prune", "reprune"):
        return "exact"      # bit copies and offsets
    if case["op"] == "lstm":
        return {"rel": 8e-7, "max": 4e-6}
    return {"rel": 1.5e-6, "max": 1e-5}
