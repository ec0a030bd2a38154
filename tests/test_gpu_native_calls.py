"""The native marshalling of the Python calls against the Python one: the same results bit for
bit for every call, with and without tensors to write into, and the same errors."""
import pytest
import torch

from paper_1811_00206_amd import binding as bs

pytestmark = pytest.mark.gpu


class _LongWay:
    """Stands in for the native module and takes nothing."""

    def __init__(self, native):
        self.stream = native.stream

    def __getattr__(self, name):
        return lambda *args: None


def _calls(bank, wide):
    g = torch.Generator(device="cuda").manual_seed(bank)
    M, K, k, N = 200, 4 * bank, bank // 4, 12
    W = torch.randn((M, K), generator=g, device="cuda")
    prune, spmv, spmm = ((bs.bs_prune_pack_wide, bs.bs_spmv_wide, bs.bs_spmm_wide) if wide else
                         (bs.bs_prune_pack, bs.bs_spmv, bs.bs_spmm))
    v, i = prune(W, bank, k)
    x, X = torch.randn(K, generator=g, device="cuda"), torch.randn((K, 2 * N), generator=g, device="cuda")
    new = lambda *s: torch.empty(s, device="cuda")
    size = bs.bs_spmm_workspace_bytes_wide if wide else bs.bs_spmm_workspace_bytes
    need = size(bs.BS_F32, M, K, bank, k, N)
    # a product of several slabs, for a workspace that the library refuses before it launches anything
    nb2 = 20000 // bank
    v2, i2 = new(M, nb2, k), torch.empty((M, nb2, k), device="cuda", dtype=i.dtype)
    X2 = new(nb2 * bank, 2 * N)
    need2 = size(bs.BS_F32, M, nb2 * bank, bank, k, 2 * N)
    assert need2 > 16
    yield "prune", lambda: prune(W, bank, k)
    yield "prune out", lambda: prune(W, bank, k, out=(torch.empty_like(v), torch.empty_like(i)))
    yield "spmv", lambda: spmv(v, i, bank, x)
    yield "spmv out", lambda: spmv(v, i, bank, x, out=new(M))
    yield "spmm", lambda: spmm(v, i, bank, X[:, :N].contiguous())
    yield "spmm slices", lambda: spmm(v, i, bank, X[:, N:], out=new(M, 3 * N)[:, N:2 * N],
                                      workspace=bs.new_spmm_workspace(need, "cuda"))
    if not wide:
        H = M // 4
        h, b, c = x[:H], torch.randn(M, generator=g, device="cuda"), torch.randn(H, generator=g, device="cuda")
        I = K - H
        Xs = torch.randn((3, I), generator=g, device="cuda")
        yield "reprune", lambda: bs.bs_reprune(v, i, bank, k // 2)
        yield "step", lambda: bs.bs_lstm_step(v, i, bank, Xs[0], h, b, c)
        yield "sequence", lambda: bs.bs_lstm_sequence(v, i, bank, Xs, h, b, c.clone())
        yield "sequence out", lambda: bs.bs_lstm_sequence(v, i, bank, Xs, h, b, c.clone(), H_all=new(3, H))
    for what, bad in (("idx type", lambda: spmv(v, i.to(torch.int32), bank, x)),
                      ("x length", lambda: spmv(v, i, bank, x[1:])),
                      ("x host", lambda: spmv(v, i, bank, x.cpu())),
                      ("bank", lambda: prune(W, 7, 2)),
                      ("k", lambda: prune(W, bank, bank + 1)),
                      ("X rows", lambda: spmm(v, i, bank, X[1:])),
                      ("X columns", lambda: spmm(v, i, bank, X.t())),
                      ("no bank", lambda: spmv(v, i, 0, x)),
                      ("workspace", lambda: spmm(v2, i2, bank, X2, workspace=bs.new_spmm_workspace(need2 - 16, "cuda")))):
        yield what, bad


def _run(call):
    try:
        out = call()
    except Exception as e:  # noqa: BLE001 - the kind and the text are what is compared
        return type(e), str(e)
    return tuple(t.cpu() for t in (out if isinstance(out, tuple) else (out,)))


@pytest.mark.parametrize("bank,wide", [(100, False), (512, True)])
def test_native_and_python_marshalling_agree(bank, wide, monkeypatch):
    names = [n for n, _ in _calls(bank, wide)]
    native = [_run(c) for _, c in _calls(bank, wide)]
    assert native[names.index("workspace")][0] is bs.BsError and "workspace" in native[names.index("workspace")][1]
    monkeypatch.setattr(bs, "_native", _LongWay(bs._native))
    for name, a, (_, call) in zip(names, native, _calls(bank, wide)):
        print("native calls", bank, name, flush=True)
        b = _run(call)
        assert len(a) == len(b), (name, a, b)
        for s, t in zip(a, b):
            assert torch.equal(s, t) if isinstance(s, torch.Tensor) else s == t, (name, s, t)
