"""The native marshalling of the Python calls (csrc/bs_calls.cpp) where the library or torch
fails.  No GPU: each test runs in a process of its own in which a stand-in for the library's
calls and for torch's current stream is loaded ahead of the real ones, on tensors that claim to
be on the GPU and lie in host memory; nothing is launched."""
import os
import subprocess
import sys
import textwrap

import pytest
import torch

from paper_1811_00206_amd import build as bs_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <ATen/ops/empty.h>
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include "bs.h"

namespace c10::hip {
HIPStream getCurrentHIPStream(DeviceIndex) {
    return HIPStream(HIPStream::UNCHECKED, Stream(Stream::DEFAULT, Device(kCUDA, 0)));
}
hipStream_t HIPStream::stream() const { return nullptr; }
}  // namespace c10::hip

// what every allocation of a tensor goes through; runs out of memory when told to
extern "C" { int out_of_memory = 0, lock_held = -1; }
namespace at::_ops {
Tensor empty_memory_format::call(c10::SymIntArrayRef size, ::std::optional<ScalarType> dtype, ::std::optional<Layout> layout,
                                 ::std::optional<Device> device, ::std::optional<bool> pin, ::std::optional<MemoryFormat> format) {
    if (out_of_memory) {
        lock_held = PyGILState_Check();
        TORCH_CHECK_WITH(OutOfMemoryError, false, "no memory left");
    }
    static const auto real = reinterpret_cast<decltype(&call)>(dlsym(
        dlopen("libtorch_cpu.so", RTLD_NOLOAD | RTLD_LAZY),
        "_ZN2at4_ops19empty_memory_format4callEN3c108ArrayRefINS2_6SymIntEEESt8optionalINS2_10ScalarTypeEES6_INS2_6"
        "LayoutEES6_INS2_6DeviceEES6_IbES6_INS2_12MemoryFormatEE"));
    return real(size, dtype, layout, device, pin, format);
}
}  // namespace at::_ops

extern "C" {
int attempts = 0, status = BS_ERR_HIP;   // of every call but the sequence
#define CALL { ++attempts; return first ? status : BS_ERR_NULL; }
int bs_spmv(const void* first, const uint8_t*, int, int64_t, int64_t, int, int, const float*, float*, void*) CALL
int bs_spmv_wide(const void* first, const uint16_t*, int, int64_t, int64_t, int, int, const float*, float*, void*) CALL
int bs_spmm(const void* first, const uint8_t*, int, int64_t, int64_t, int, int, const float*, int64_t, int64_t, float*,
            int64_t, void*, size_t, void*) CALL
int bs_spmm_wide(const void* first, const uint16_t*, int, int64_t, int64_t, int, int, const float*, int64_t, int64_t, float*,
                 int64_t, void*, size_t, void*) CALL
int bs_prune_pack(const void* first, int, int64_t, int64_t, int, int, void*, uint8_t*, void*) CALL
int bs_prune_pack_wide(const void* first, int, int64_t, int64_t, int, int, void*, uint16_t*, void*) CALL
int bs_reprune(const void* first, const uint8_t*, int, int64_t, int64_t, int, int, int, void*, uint8_t*, void*) CALL
// advances the cell state step by step; the first attempt fails at its second step
int bs_lstm_sequence(const void*, const uint8_t*, int, int64_t, int64_t, int, int, const float*, int64_t T,
                     const float*, const float*, float* c, float*, void*) {
    const int attempt = ++attempts;
    for (int64_t t = 0; t < T; ++t) {
        if (attempt == 1 && t == 1) return BS_ERR_HIP;
        c[0] += 1.f;
    }
    return BS_OK;
}
}
"""

PREAMBLE = """
    import ctypes, os, sys
    import torch
    stand_in = ctypes.CDLL(os.environ["BS_STAND_IN"], mode=ctypes.RTLD_GLOBAL)
    from paper_1811_00206_amd import binding as bs

    attempts = ctypes.c_int.in_dll(stand_in, "attempts")

    class Library:
        '''The ctypes library: host-only queries are the real ones, other calls count as attempts.'''
        def __init__(self, lib):
            self.lib = lib
        def __getattr__(self, name):
            if name in ("bs_status_str", "bs_spmm_workspace_bytes", "bs_spmm_workspace_bytes_wide"):
                return getattr(self.lib, name)
            def call(*args):
                attempts.value += 1
                return 0
            return call

    bs._lib = Library(bs.load_library())
    kept = []

    def gpu(*size, dtype=torch.float32):
        '''zeros in host memory that claim to be on the GPU'''
        host = torch.zeros(size, dtype=dtype)
        kept.append(host)
        nbytes, dev = host.numel() * host.element_size(), torch.device("cuda", 0)
        storage = torch._C._construct_storage_from_data_pointer(host.data_ptr(), dev, nbytes)
        return torch._C._construct_CUDA_Tensor_From_Storage_And_Metadata(
            dict(size=tuple(size), stride=host.stride(), dtype=dtype, storage_offset=0), storage)
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("stand_in")
    src, lib = str(tmp / "stand_in.cpp"), str(tmp / "stand_in.so")
    with open(src, "w") as f:
        f.write(STAND_IN)
    subprocess.check_call([*bs_build.native_compiler(), "-I" + os.path.join(ROOT, "include"), "-shared", "-o", lib, src,
                           "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-lc10", "-lc10_hip",
                           "-ltorch_cpu"])
    return lib


# calls whose results the native code allocates: name -> call
ALLOCATING = """
    M, bank, nb, k, N = 4, 8, 2, 4, 3
    v, i, W = gpu(M, nb, k), gpu(M, nb, k, dtype=torch.uint8), gpu(M, nb * bank)
    x, X = gpu(nb * bank), gpu(nb * bank, N)
    x4, b, h, c, X4 = gpu(15), gpu(4), gpu(1), gpu(1), gpu(2, 15)
    allocating = {"spmv": lambda: bs.bs_spmv(v, i, bank, x), "spmm": lambda: bs.bs_spmm(v, i, bank, X),
                  "prune": lambda: bs.bs_prune_pack(W, bank, k), "reprune": lambda: bs.bs_reprune(v, i, bank, k),
                  "step": lambda: bs.bs_lstm_step(v, i, bank, x4, h, b, c),
                  "sequence": lambda: bs.bs_lstm_sequence(v, i, bank, X4, h, b, c)}
"""


def _run(stand_in, body):
    code = textwrap.dedent(PREAMBLE + ALLOCATING) + textwrap.dedent(body)
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env={**os.environ, "BS_STAND_IN": stand_in},
                         capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr


def test_a_sequence_that_fails_at_a_later_step_is_not_tried_again(stand_in):
    """By the second step the cell state has advanced in place: a second attempt would start
    from it and return wrong states without an error."""
    _run(stand_in, """
        H, I, T, bank, k = 8, 8, 3, 4, 2
        v, i = gpu(4 * H, 4, k), gpu(4 * H, 4, k, dtype=torch.uint8)
        c = gpu(H)
        try:
            bs.bs_lstm_sequence(v, i, bank, gpu(T, I), gpu(H), gpu(4 * H), c, H_all=gpu(T, H))
        except bs.BsError as e:
            assert e.status == 5 and "bs_lstm_sequence" in str(e), e
        else:
            raise AssertionError("no error")
        assert attempts.value == 1, attempts.value
        assert ctypes.c_float.from_address(c.data_ptr()).value == 1.0
    """)


def test_a_status_is_raised_after_one_attempt(stand_in):
    _run(stand_in, """
        M, bank, nb, k, N = 4, 8, 2, 4, 3
        for wide in (False, True):
            off = torch.uint16 if wide else torch.uint8
            v, i, W = gpu(M, nb, k), gpu(M, nb, k, dtype=off), gpu(M, nb * bank)
            tail = "_wide" if wide else ""
            call = lambda name: getattr(bs, name + tail)
            calls = {"bs_spmv": lambda: call("bs_spmv")(v, i, bank, gpu(nb * bank), out=gpu(M)),
                     "bs_spmm": lambda: call("bs_spmm")(v, i, bank, gpu(nb * bank, N), out=gpu(M, N)),
                     "bs_prune_pack": lambda: call("bs_prune_pack")(W, bank, k, out=(v, i))}
            if not wide:
                calls["bs_reprune"] = lambda: bs.bs_reprune(v, i, bank, k, out=(gpu(M, nb, k), i))
            for name, f in calls.items():
                for status in range(1, 9):
                    ctypes.c_int.in_dll(stand_in, "status").value = status
                    attempts.value = 0
                    try:
                        f()
                    except bs.BsError as e:
                        assert e.status == status and str(e).startswith(name + tail + ":"), (name, e)
                    else:
                        raise AssertionError(name + ": no error")
                    assert attempts.value == 1, (name, status, attempts.value)
    """)


def test_exceptions_keep_their_types(stand_in):
    """Out of memory, as the allocator reports it, is torch.OutOfMemoryError; what a dispatch
    mode raises is what the caller sees."""
    _run(stand_in, """
        from torch.utils._python_dispatch import TorchDispatchMode

        class Refuses(TorchDispatchMode):
            def __torch_dispatch__(self, func, types, args=(), kwargs=None):
                raise KeyError("refused")

        fails = ctypes.c_int.in_dll(stand_in, "out_of_memory")
        for name, f in allocating.items():
            for want, text in ((KeyError, "refused"), (torch.OutOfMemoryError, "no memory left")):
                fails.value = want is not KeyError
                try:
                    if want is KeyError:
                        with Refuses():
                            f()
                    else:
                        f()
                except Exception as e:
                    assert type(e) is want and text in str(e), (name, type(e), e)
                else:
                    raise AssertionError(name + ": no error")
        assert attempts.value == 0
    """)


def test_allocations_give_the_interpreter_lock_up(stand_in):
    _run(stand_in, """
        ctypes.c_int.in_dll(stand_in, "out_of_memory").value = 1
        held = ctypes.c_int.in_dll(stand_in, "lock_held")
        for name, f in allocating.items():
            held.value = -1
            try:
                f()
            except torch.OutOfMemoryError:
                pass
            assert held.value == 0, (name, held.value)
    """)


def test_outputs_that_are_too_small_are_refused(stand_in):
    """Refused before any call; a larger output is written at its start, as ever."""
    _run(stand_in, """
        H, I, T, bank, k = 8, 8, 3, 4, 2
        v, i = gpu(4 * H, 4, k), gpu(4 * H, 4, k, dtype=torch.uint8)
        X, h, b, c = gpu(T, I), gpu(H), gpu(4 * H), gpu(H)
        W = gpu(H, I)
        calls = {"H_all": (T * H, lambda t: bs.bs_lstm_sequence(v, i, bank, X, h, b, c, H_all=t)),
                 "c_out": (H, lambda t: bs.bs_lstm_step(v, i, bank, h, h, b, c, c_out=t, h_out=gpu(H))),
                 "h_out": (H, lambda t: bs.bs_lstm_step(v, i, bank, h, h, b, c, c_out=c, h_out=t)),
                 "gemv": (H, lambda t: bs.bs_dense_gemv(W, h, out=t)),
                 "gemm": (H * 2, lambda t: bs.bs_dense_gemm(W, gpu(I, 2), out=t))}
        ctypes.c_int.in_dll(stand_in, "status").value = 0
        for name, (n, f) in calls.items():
            attempts.value = 1       # the stand-in's sequence fails at its first attempt only
            try:
                f(gpu(n - 1))
            except ValueError as e:
                assert str(n) in str(e), e
            else:
                raise AssertionError(name + ": no error")
            assert attempts.value == 1, name
            for room in (n, n + 1):
                f(gpu(room))
            assert attempts.value == 3, name
    """)


def test_a_workspace_in_host_memory_is_refused(stand_in):
    """The kernels write to it.  Where a product needs none, none is looked at."""
    _run(stand_in, """
        ctypes.c_int.in_dll(stand_in, "status").value = 0
        M, N = 200, 24
        for wide, bank, k, nb, spmm, size in ((False, 100, 10, 200, bs.bs_spmm, bs.bs_spmm_workspace_bytes),
                                              (True, 512, 16, 40, bs.bs_spmm_wide, bs.bs_spmm_workspace_bytes_wide)):
            for nb_ in (nb, 1):
                need = size(bs.BS_F32, M, nb_ * bank, bank, k, N)
                assert (need > 0) == (nb_ > 1)
                v, X = gpu(M, nb_, k), gpu(nb_ * bank, N)
                i, Y = gpu(M, nb_, k, dtype=torch.uint16 if wide else torch.uint8), gpu(M, N)
                for host in (torch.empty(max(need, 16), dtype=torch.uint8), bytearray(max(need, 16))):
                    attempts.value = 0
                    if not need and not isinstance(host, torch.Tensor):
                        continue
                    try:
                        spmm(v, i, bank, X, out=Y, workspace=host)
                    except TypeError as e:
                        assert need and "workspace" in str(e), e
                    else:
                        assert not need
                    assert attempts.value == (0 if need else 1)
    """)


def test_tensors_without_memory_raise(stand_in):
    """Tensors of a transform have no address to ask for and raise, with the interpreter lock held;
    fake ones have a null one, which the library refuses."""
    _run(stand_in, """
        import warnings
        from torch._subclasses.fake_tensor import FakeTensorMode
        warnings.simplefilter("ignore")      # torch's own, about addresses of fake tensors
        M, bank, nb, k, N = 8, 16, 4, 4, 3
        K, H, T = nb * bank, M // 4, 3
        i, iw = gpu(M, nb, k, dtype=torch.uint8), gpu(M, nb, k, dtype=torch.uint16)

        def calls(v, x, X, W, Xs, h, b):
            y, Y, out = gpu(M), gpu(M, N), (gpu(M, nb, k), i)
            return {"bs_spmv": lambda: bs.bs_spmv(v, i, bank, x, out=y),
                    "bs_spmv_wide": lambda: bs.bs_spmv_wide(v, iw, bank, x, out=y),
                    "bs_spmm": lambda: bs.bs_spmm(v, i, bank, X, out=Y),
                    "bs_prune_pack": lambda: bs.bs_prune_pack(W, bank, k, out=out),
                    "bs_reprune": lambda: bs.bs_reprune(v, i, bank, k, out=out),
                    "bs_lstm_sequence": lambda: bs.bs_lstm_sequence(v, i, bank, Xs, h, b, h, H_all=gpu(T, H))}

        sizes = ((M, nb, k), (K,), (K, N), (M, K), (T, K - H), (H,), (M,))
        refused = {}

        def of_a_transform(*tensors):
            for name, f in calls(*tensors).items():
                try:
                    f()
                except RuntimeError as e:
                    refused[name] = str(e)
            return tensors[0]

        torch.func.vmap(of_a_transform)(*(gpu(2, *s) for s in sizes))
        assert len(refused) == 6 and all("data pointer" in e for e in refused.values()), refused
        assert attempts.value == 0

        with FakeTensorMode():
            fake = [torch.empty(s, device="cuda") for s in sizes]
        for name, f in calls(*fake).items():
            if name == "bs_lstm_sequence":    # the stand-in's takes no notice of its pointers
                continue
            attempts.value = 0
            try:
                f()
            except bs.BsError as e:
                assert e.status == 1 and attempts.value == 1, (name, e, attempts.value)
            else:
                raise AssertionError(name + ": no error")
    """)
