"""The calls that go through the native module: the same outputs as through the Python function's own checks and ctypes, the given
outputs and streams used, and everything that is refused refused in the same way."""
import types

import pytest
import torch

import paper_2505_18663_amd as dvdq

pytestmark = pytest.mark.gpu

M, K, N = 70, 512, 264


@pytest.fixture
def both(monkeypatch):
    """call(f) -> (f() through the native module, f() without it)"""
    dvdq.lib()
    assert dvdq._marshal.__file__ == dvdq._MARSHAL_PATH   # (else both would go through ctypes)
    refuse = types.SimpleNamespace(**{f: lambda *a: None for f in ("qlinear", "rotate_quant", "rotate_quant_blockwise", "w4ax_gemm",
                                                                  "gbs_reset", "gbs_step")})
    native = dvdq._marshal

    def call(f):
        monkeypatch.setattr(dvdq, "_marshal", native)
        first = f()
        monkeypatch.setattr(dvdq, "_marshal", refuse)
        return first, f()
    return call


def _inputs(fmt):
    g = torch.Generator(device="cuda").manual_seed(5)
    packed = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    w, layout = {"int8": (dvdq.w4_prepack, dvdq.W_NATIVE), "packed4": (dvdq.w4_prepack, dvdq.W_NATIVE),
                 "fp6": (dvdq.w4_prepack_fp6, dvdq.W_NATIVE_FP6), "canonical": (lambda t: t, dvdq.W_CANONICAL)}[fmt]
    codes = {"packed4": dvdq.CODES_PACKED4, "fp6": dvdq.CODES_FP6}.get(fmt, dvdq.CODES_INT8)
    zero = None if fmt == "canonical" else torch.randint(-8, 8, (N,), generator=g, device="cuda", dtype=torch.int8)
    return {"x": torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16), "w": w(packed), "layout": layout, "codes": codes,
            "ws": torch.rand((N,), generator=g, device="cuda"), "z": zero, "b": torch.randn((N,), device="cuda").to(torch.bfloat16)}


def _equal(a, b):
    if isinstance(a, tuple):
        assert type(a) is type(b) and len(a) == len(b)
        for x, y in zip(a, b):
            _equal(x, y)
    else:
        assert a.shape == b.shape and a.dtype == b.dtype and a.device == b.device and torch.equal(a, b)


@pytest.mark.parametrize("fmt", ["int8", "packed4", "fp6", "canonical"])
def test_same_outputs(fmt, both):
    i = _inputs(fmt)
    bits = 4 if fmt in ("packed4", "fp6") else 8
    sums = i["z"] is not None
    a, b = both(lambda: dvdq.rotate_quant(i["x"], 128, bits, codes_format=i["codes"], want_rowsum=sums))
    _equal(a[1:], b[1:])
    if fmt != "fp6":   # (the container's rows past M are not written)
        _equal(a[0], b[0])
    gemm = lambda y=None: dvdq.w4ax_gemm(a[0], a[1], i["w"], i["ws"], bits, i["layout"], bias=i["b"], y=y, codes_format=i["codes"],
                                         w_zero=i["z"], code_rowsum=a[2] if sums else None, K=K)
    _equal(*both(gemm))
    y = torch.empty((M, N), device="cuda", dtype=torch.bfloat16)
    assert all(r is y for r in both(lambda: gemm(y)))
    layer = lambda **k: dvdq.qlinear(i["x"], i["w"], i["ws"], 128, bits, i["layout"], bias=i["b"], codes_format=i["codes"], w_zero=i["z"], **k)
    p, q = both(layer)
    _equal(p[0], q[0])
    assert p[1].shape == q[1].shape
    workspace = torch.empty_like(p[1])
    assert all(r[0] is y and r[1] is workspace for r in both(lambda: layer(y=y, workspace=workspace)))
    _equal(y, p[0])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = layer(stream=side)[0]
    side.synchronize()
    _equal(got, y)


def test_blockwise_and_controller(both):
    i = _inputs("int8")
    for sums in (False, True):
        _equal(*both(lambda: dvdq.rotate_quant_blockwise(i["x"], 128, 4, 256, want_rowsum=sums)))
    f = torch.randn((3, 5000), device="cuda").to(torch.bfloat16)

    def run():
        ctl = dvdq.GbsController(0.5)
        ctl.step(f[1], f[0])
        ctl.step(f[2], f[1])
        return ctl.read()
    a, b = both(run)
    assert a == b


def test_refused_in_the_same_way(both):
    i = _inputs("int8")
    x, w, ws = i["x"], i["w"], i["ws"]
    codes, scale = dvdq.rotate_quant(x, 128, 8)
    calls = [lambda: dvdq.qlinear(x.float(), w, ws, 128, 8, dvdq.W_NATIVE), lambda: dvdq.qlinear(x.cpu(), w, ws, 128, 8, dvdq.W_NATIVE),
             lambda: dvdq.qlinear(x.t(), w, ws, 128, 8, dvdq.W_NATIVE), lambda: dvdq.qlinear(x, w[:-256], ws, 128, 8, dvdq.W_NATIVE),
             lambda: dvdq.qlinear(x, w, ws, 96, 8, dvdq.W_NATIVE), lambda: dvdq.qlinear(x, w, ws, 128, 7, dvdq.W_NATIVE),
             lambda: dvdq.qlinear(x, w, ws, 128, 8, 9), lambda: dvdq.qlinear(x, w, ws, 128, 8, dvdq.W_NATIVE, bias=i["b"][1:]),
             lambda: dvdq.qlinear(x, w, ws, 128, 8, dvdq.W_NATIVE, workspace=torch.empty(256, dtype=torch.uint8, device="cuda")),
             lambda: dvdq.qlinear(x[:0], w, ws, 128, 8, dvdq.W_NATIVE), lambda: dvdq.qlinear(x, w, ws, 128.0, 8, dvdq.W_NATIVE),
             lambda: dvdq.rotate_quant(x, 128, 8, codes=codes[1:]), lambda: dvdq.rotate_quant(x, 128, 6, codes_format=dvdq.CODES_FP6),
             lambda: dvdq.w4ax_gemm(codes, scale, w, ws, 8, dvdq.W_NATIVE, w_zero=i["z"]),
             lambda: dvdq.w4ax_gemm(codes, scale[1:], w, ws, 8, dvdq.W_NATIVE), lambda: dvdq.w4ax_gemm(codes, scale, None, ws, 8, dvdq.W_NATIVE),
             lambda: dvdq.rotate_quant_blockwise(x, 128, 4, 100), lambda: dvdq.GbsController(0.1).step(x, x[1:])]
    for f in calls:
        def kind():
            try:
                f()
            except Exception as e:
                return type(e), getattr(e, "status", None), str(e)
        a, b = both(kind)
        assert a is not None and a == b
