"""What the native marshalling hands to the C entry points and what it refuses, without a GPU: the GEMMs' entry points are replaced by
functions that record their arguments and return the library's status for a missing buffer."""
import ctypes as C
import dataclasses
import sys
import types

import pytest
import torch

import paper_2605_21072_amd as q
from paper_2605_21072_amd import binding

_VP, _I32, _I64 = C.c_void_p, C.c_int32, C.c_int64
_OPERANDS = [_VP, _I64, _VP, _VP, _I64, _VP, _VP, _VP, _I32, _I32, _I32, _I32]     # Xq, ldxq, s_x, Wq, ldwq, s_n, s_o, bias, M, N, K, K_o


@pytest.fixture
def no_stream(monkeypatch):
    """The current stream's handle without a device to have one."""
    if not q.lib_path().exists():
        from paper_2605_21072_amd import build
        build.build()
    binding._load_host(q.load_library())
    monkeypatch.setattr(binding, "_stream", lambda stream: 0)


@pytest.fixture
def gemm_calls(no_stream):
    """The arguments of each GEMM call behind the name of its entry point."""
    calls = []

    def status(*args):
        calls.append(args)
        return 0 if all(args[i] for i in (1, 3, 4, 6, 7)) else -1

    w8 = C.CFUNCTYPE(C.c_int, _I32, *_OPERANDS, _VP, C.c_int, _I64, _VP, _VP, _VP)(lambda variant, *a: status("w8", *a))
    w4 = C.CFUNCTYPE(C.c_int, *_OPERANDS, _VP, C.c_int, _I64, _VP, _VP, _I32, _VP)(lambda *a: status("w4", *a))
    q8 = C.CFUNCTYPE(C.c_int, *_OPERANDS, C.c_int, C.c_float, _VP, _I64, _I32, _VP)(lambda *a: status("q8", *a))
    lib = q.load_library()
    real = [C.cast(f, _VP).value for f in (lib.qarvd_linear, lib.qarvd_linear_workspace, lib.qarvd_packed_ld, lib.qarvd_quant_act,
                                           lib.qarvd_quant_act_static)]
    binding._host.init(real + [C.cast(f, _VP).value for f in (w8, w4, q8)])
    yield calls
    binding._load_host(lib)


def _layer(bits=8):
    w = torch.zeros((16, 256), dtype=torch.int8)
    return q.DualScaleWeight(w, torch.ones(16), torch.ones(16), None, 0, 16, 128, None, bits), torch.zeros((4, 256), dtype=torch.int8), torch.ones(4)


def test_a_static_scale_that_is_no_number_is_refused(no_stream):
    X = torch.zeros((4, 128))
    for scale in (None, "0.1", [0.1]):
        with pytest.raises(TypeError):
            q.quant_act_static(X, None, 0, scale)


@pytest.mark.parametrize("bits", [8, 4])
def test_out_dtype_is_torchs_default_or_of_no_matter_beside_Y(gemm_calls, bits):
    w, Xq, s_x = _layer(bits)
    assert q.w8a8_dual_gemm(Xq, s_x, w, None, 4, out_dtype=None).dtype == torch.get_default_dtype() == torch.float32
    assert q.w8a8_dual_gemm(Xq, s_x, w, None, 4).dtype == torch.bfloat16
    for dtype in (None, "bf16", torch.float16):
        Y = torch.zeros((4, 16), dtype=torch.bfloat16)
        assert q.w8a8_dual_gemm(Xq, s_x, w, None, 4, out_dtype=dtype, Y=Y) is Y
        assert gemm_calls[-1][13:16] == (Y.data_ptr(), 1, 16)
    for dtype in (torch.float16, "bf16"):
        with pytest.raises(TypeError):
            q.w8a8_dual_gemm(Xq, s_x, w, None, 4, out_dtype=dtype)


def test_a_missing_vector_is_refused_by_the_entry_point(gemm_calls):
    w, Xq, s_x = _layer()
    Y8 = torch.zeros((4, 16), dtype=torch.int8)
    for missing in ("s_x", "s_normal", "s_outlier"):
        wm = w if missing == "s_x" else dataclasses.replace(w, **{missing: None})
        sm = None if missing == "s_x" else s_x
        for call in (lambda: q.w8a8_dual_gemm(Xq, sm, wm, None, 4), lambda: q.w8a8_dual_gemm_q8(Xq, sm, wm, None, 4, 0.1, Y8=Y8)):
            with pytest.raises(q.QarvdError) as e:
                call()
            assert e.value.status == -1
    assert q.w8a8_dual_gemm_q8(Xq, s_x, w, None, 4, 0.1, Y8=Y8) is Y8 and gemm_calls[-1][15] == Y8.data_ptr()


def test_only_the_online_calls_need_the_module_and_say_how_to_get_it(no_stream, monkeypatch):
    w, Xq, s_x = _layer()
    for other in (None, types.SimpleNamespace(__file__="_host.so", torch_version="1.0")):        # absent; built for another torch
        monkeypatch.setattr(binding, "_lib", None)
        monkeypatch.setattr(binding, "_host", None)
        monkeypatch.delattr(q, "_host", raising=False)          # (`from . import` looks for the attribute first)
        monkeypatch.setitem(sys.modules, q.__name__ + "._host", other)
        assert q.packed_k(1536, 0) == 1536 and q.quantize_weight_workspace(16, 1536) > 0
        for call in (lambda: q.w8a8_linear(s_x, w, None), lambda: q.quant_act(s_x, None, 0), lambda: q.w8a8_dual_gemm(Xq, s_x, w, None, 4)):
            with pytest.raises(ImportError, match="paper_2605_21072_amd.build"):
                call()
