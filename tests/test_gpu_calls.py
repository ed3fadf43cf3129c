"""The extension module's calls against the general path of the binding: same results over the forms of arguments that
both take, same errors for those that neither does."""
import ctypes
import importlib
import os
import shutil
import subprocess
import sys
import types

import pytest
import torch

from paper_2603_05232_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _none(*args):
    return None


GENERAL = types.SimpleNamespace(act_lift_quant=_none, slide_sparse_gemm=_none, slide_sparse_gemm_fused=_none)


def _both(monkeypatch, f):
    """f() through the extension module (which must have taken the call) and through the general path."""
    binding.load()
    taken = []
    real = binding._calls

    def spy(name):
        def call(*args):
            r = getattr(real, name)(*args)
            taken.append(r is not None)
            return r
        return call

    monkeypatch.setattr(binding, "_calls", types.SimpleNamespace(**{n: spy(n) for n in vars(GENERAL)}))
    a = f()
    assert taken and all(taken)
    monkeypatch.setattr(binding, "_calls", GENERAL)
    b = f()
    monkeypatch.undo()
    return a, b


def _same(a, b):
    assert type(a) is type(b)
    if isinstance(a, tuple):
        assert len(a) == len(b)
        for x, y in zip(a, b):
            _same(x, y)
    elif a is not None:
        assert a.shape == b.shape and a.dtype == b.dtype and a.stride() == b.stride() and a.device == b.device
        assert torch.equal(a.view(torch.uint8) if a.element_size() == 1 else a.view(torch.int16), b.view(torch.uint8) if b.element_size() == 1 else b.view(torch.int16))


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("src", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,N", [(0, 4), (1, 2), (5, 4), (3, 8)])
def test_quantisation(monkeypatch, dtype, src, M, N):
    X = torch.randn((M, 200), device=DEV).to(src)
    for x in (X, X[:, :131], X[:1, ::1], torch.nn.Parameter(X)):
        _same(*_both(monkeypatch, lambda: binding.act_lift_quant(x, N, dtype)))
    out = torch.zeros((M, binding.slide_lifted_ld(200, N, dtype)), dtype=binding._STORAGE_DTYPE[dtype], device=DEV)
    s_x = torch.zeros((M,), device=DEV)
    a, b = _both(monkeypatch, lambda: binding.act_lift_quant(X, N, dtype, out=out, s_x=s_x))
    assert a[0] is out and b[0] is out and a[1] is s_x and b[1] is s_x


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("M", [1, 9, 130])
def test_gemms(monkeypatch, dtype, M):
    O, K = 264, 512
    Wq, s_w = binding.slide_prune_quant(torch.randn((O, K), device=DEV), 4, dtype)
    X = torch.randn((M, K), device=DEV)
    XL, s_x = binding.act_lift_quant(X, 4, dtype)
    wv, wm = binding.slide_decompose(Wq, 4, dtype)
    ws = torch.empty((max(16, binding.slide_gemm_workspace_bytes(M, O, XL.shape[1], dtype)),), dtype=torch.uint8, device=DEV)
    wide = torch.zeros((M, O + 8), dtype=torch.bfloat16, device=DEV)
    for out in (None, wide[:, :O]):
        for w in (None, ws, ws.view(torch.int32)):
            a, b = _both(monkeypatch, lambda: binding.slide_sparse_gemm(XL, s_x, wv, wm, s_w, O, dtype, out=out, workspace=w).clone())
            _same(a, b)
    Xq, s_x = binding.act_lift_quant(X, 2, dtype)
    fv, fm = binding.slide_decompose_fused(Wq, 4, dtype)
    wide_x = torch.zeros((M, K + 64), dtype=Xq.dtype, device=DEV)
    wide_x[:, :K] = Xq[:, :K]
    for x in (Xq, wide_x):
        for out in (None, wide[:, :O]):
            for w in (None, ws):
                a, b = _both(monkeypatch, lambda: binding.slide_sparse_gemm_fused(x, s_x, fv, fm, s_w, O, K, 4, dtype, out=out, workspace=w).clone())
                _same(a, b)


def test_refused_calls_raise_as_before():
    X = torch.randn((4, 256), device=DEV)
    Xq, s_x = binding.act_lift_quant(X, 2, "i8")
    w = torch.zeros((128 * 256,), dtype=torch.uint8, device=DEV)
    s_w = torch.ones((128,), device=DEV)
    for f, error in ((lambda: binding.act_lift_quant(X, 9, "i8"), binding.SlideSparseError), (lambda: binding.act_lift_quant(X, 4, "i4"), KeyError),
                     (lambda: binding.act_lift_quant(X.half(), 4, "i8"), TypeError), (lambda: binding.act_lift_quant(X.T, 4, "i8"), AssertionError),
                     (lambda: binding.act_lift_quant(X.cpu(), 4, "i8"), AssertionError), (lambda: binding.act_lift_quant(X[0], 4, "i8"), ValueError),
                     (lambda: binding.slide_sparse_gemm(Xq[:, :100].contiguous(), s_x, w, w, s_w, 128, "i8"), binding.SlideSparseError),
                     (lambda: binding.slide_sparse_gemm(Xq, s_x, w, None, s_w, 128, "i8"), binding.SlideSparseError),
                     (lambda: binding.slide_sparse_gemm_fused(Xq, None, w, w, s_w, 128, 256, 4, "i8"), binding.SlideSparseError),
                     (lambda: binding.slide_sparse_gemm_fused(Xq, s_x, w, w, s_w, 128, 256, 5, "i8"), binding.SlideSparseError),
                     (lambda: binding.slide_sparse_gemm_fused(Xq, s_x, w, w, s_w, 128, 512, 4, "i8"), AssertionError),
                     (lambda: binding.slide_sparse_gemm_fused(Xq, s_x, w, w, s_w, 128, 256, 4, "i8", workspace=w[1:]), binding.SlideSparseError)):
        with pytest.raises(error):
            f()


STUB = """
#include <stdint.h>
extern "C" {{
int calls = 0;
{}
int64_t slide_lifted_ld(int64_t, int, int) {{ return 128; }}
const char* ss_status_string(int) {{ return "stub"; }}
int act_lift_quant() {{ return ++calls == 1 ? 6 : 0; }}
int slide_sparse_gemm_ws() {{ return ++calls == 1 ? 6 : 0; }}
int slide_sparse_gemm_fused_ws() {{ return ++calls == 1 ? 6 : 0; }}
}}
"""


@pytest.fixture(scope="module")
def failing_copy(tmp_path_factory):
    """The binding of a copy of the package whose library reports a HIP error (6) for the first launch and none for the next."""
    root = tmp_path_factory.mktemp("copy")
    shutil.copytree(os.path.dirname(binding.LIB_PATH), root / "failing_copy", ignore=shutil.ignore_patterns("csrc", "__pycache__", "lib*.so"))
    own = ("slide_lifted_ld", "ss_status_string", "act_lift_quant", "slide_sparse_gemm_ws", "slide_sparse_gemm_fused_ws")
    (root / "stub.cpp").write_text(STUB.format("\n".join(f"int {n}() {{ return 0; }}" for n in binding.EXPORTS if n not in own)))
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(root / "failing_copy" / "libslidesparse.so"), str(root / "stub.cpp")], check=True)
    sys.path.insert(0, str(root))
    try:
        yield importlib.import_module("failing_copy.binding")
    finally:
        sys.path.remove(str(root))


@pytest.mark.parametrize("call", ["act_lift_quant", "slide_sparse_gemm_ws", "slide_sparse_gemm_fused_ws"])
def test_a_launch_error_raises_and_is_not_tried_again(failing_copy, call):
    calls = ctypes.c_int.in_dll(failing_copy.load(), "calls")
    calls.value = 0
    X = torch.zeros((4, 128), device=DEV)
    q, s, w = X.to(torch.int8), X[:, 0].contiguous(), torch.zeros((64,), dtype=torch.uint8, device=DEV)
    f = {"act_lift_quant": lambda: failing_copy.act_lift_quant(X, 2, "i8"),
         "slide_sparse_gemm_ws": lambda: failing_copy.slide_sparse_gemm(q, s, w, w, s, 4, "i8", workspace=w),
         "slide_sparse_gemm_fused_ws": lambda: failing_copy.slide_sparse_gemm_fused(q, s, w, w, s, 4, 128, 4, "i8", workspace=w)}[call]
    with pytest.raises(failing_copy.SlideSparseError, match=call) as e:
        f()
    assert e.value.code == 6 and calls.value == 1
    f()
    assert calls.value == 2
