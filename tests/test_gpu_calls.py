"""The binding's native calls give what its Python code gives: outputs, returned objects and refusals.  Every call below runs
through both, on its own copies of the inputs."""
import ctypes as C
import types

import numpy as np
import pytest
import torch

import paper_2511_05811_amd as moss
from paper_2511_05811_amd import binding, build

ROW, COL = moss.MOSS_Q_ROW, moss.MOSS_Q_COL


def both(monkeypatch, call):
    """call() through the native calls and through the Python code: (value or exception type) of each"""
    got = []
    for native in (True, False):
        monkeypatch.setattr(binding, "_calls", None if native else False)
        try:
            got.append(call())
        except Exception as e:                       # noqa: BLE001  (which one is the result)
            got.append(type(e))
    return got


def same(a, b):
    if isinstance(a, dict):
        assert list(a) == list(b)
        for k in a:
            same(a[k], b[k])
    elif isinstance(a, (tuple, list)):
        assert len(a) == len(b)
        for x, y in zip(a, b):
            same(x, y)
    elif isinstance(a, torch.Tensor):
        assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.device == b.device and torch.equal(a, b)
    else:
        assert a is b


def test_plain_arguments_are_what_the_native_calls_take():
    """On the CPU nothing is plain: every function answers None, and the Python code refuses what it always refused."""
    binding._bind_calls()
    if not binding._calls:
        pytest.fail("_moss_calls has not been built for this torch")
    x = torch.zeros(4, 64, dtype=torch.bfloat16)
    assert binding._calls.quant_act_2level(x, ROW, None, None) is None
    assert binding._calls.swiglu_bf16(x, x, None, None) is None
    assert binding._calls.gemm_fp8_mx(x, None, x, x, None, x, None, False) is None
    with pytest.raises(AssertionError):
        moss.quant_act_2level(x)


@pytest.mark.parametrize("other", ["torch_version", "interface", "interface of no build"])
def test_native_calls_built_for_another_torch_or_library_are_left_alone(monkeypatch, other):
    """They would read tensors of another layout, or call the library by another signature."""
    lib = moss.load()
    lib.moss_internal_interface.restype = C.c_uint32
    marks = dict(torch_version=torch.__version__, interface=lib.moss_internal_interface())
    bound = []
    fake = types.SimpleNamespace(bind=lambda *a: bound.append(a), **marks)
    monkeypatch.setattr(moss, "_moss_calls", fake, raising=False)
    monkeypatch.setattr(binding, "_calls", None)
    assert binding._bind_calls() is fake and len(bound) == 1            # (the marks as they are)
    for name, value in {"torch_version": dict(torch_version="1.0"), "interface": dict(interface=marks["interface"] ^ 2),
                        "interface of no build": dict(interface=0)}[other].items():
        setattr(fake, name, value)
    assert binding._bind_calls() is False and len(bound) == 1


def test_the_library_builds_without_what_the_native_calls_need(monkeypatch, tmp_path, capsys):
    lib, calls = tmp_path / "lib.so", tmp_path / "calls.so"
    calls.write_text("of an earlier build")
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "CALLS", str(calls))
    monkeypatch.setattr(build, "SOURCES", ["moss_api.hip"])
    monkeypatch.setenv("CXX", str(tmp_path / "no compiler here"))
    assert build.build() == str(lib)
    assert lib.exists() and not calls.exists() and "no native calls" in capsys.readouterr().err


@pytest.fixture
def data():
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    r = lambda *s, k=1.0: torch.randn(*s, generator=gen, device="cuda:0") * k
    return dict(x=r(64, 256).bfloat16(), wide=r(64, 320).bfloat16()[:, :256], w=r(96, 256, k=0.02), gamma=r(256).bfloat16(), g=r(96, 256, k=1e-3),
                y=r(64, 256).bfloat16())


def adamw(t=1):
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.95))
    return moss.AdamWArgs(3e-4, 0.9, 0.95, 1e-8, 0.1, 1.0 - b1, 1.0 - b2, 1.0 - b1 ** t, 1.0 - b2 ** t, 1.0, 500, t)


def quantized(d):
    q = moss.quant_act_2level(d["x"], ROW)
    w, s = torch.randint(0, 120, (96, 256), device="cuda:0", dtype=torch.uint8, generator=torch.Generator("cuda:0").manual_seed(1)), q["s"]
    return q, w, s


CALLS = {
    "rows": lambda d: moss.quant_act_2level(d["x"], ROW),
    "both groupings, strided": lambda d: moss.quant_act_2level(d["wide"], ROW | COL | moss.MOSS_EXP_CEIL),
    "outputs and scratch given": lambda d: moss.quant_act_2level(d["x"], COL, out=dict(moss.quant_act_2level(d["x"], ROW | COL)),
                                                                 workspace=torch.zeros(16384, dtype=torch.uint8, device="cuda:0")),
    "scale given": lambda d: moss.quant_act_2level(d["x"], ROW, out=dict(s=torch.zeros(1, device="cuda:0"))),
    "codes without exponents": lambda d: moss.quant_act_2level(d["x"], ROW, out=dict(q_row=torch.zeros(64, 256, dtype=torch.uint8, device="cuda:0"))),
    "no grouping": lambda d: moss.quant_act_2level(d["x"], 0),
    "unknown flag": lambda d: moss.quant_act_2level(d["x"], 64),
    "three dimensions": lambda d: moss.quant_act_2level(d["x"][None], ROW),
    "float32": lambda d: moss.quant_act_2level(d["x"].float(), ROW),
    "transposed": lambda d: moss.quant_act_2level(d["x"].t(), ROW),
    "not a tensor": lambda d: moss.quant_act_2level(None, ROW),
    "odd width": lambda d: moss.quant_act_2level(d["x"][:, :40], ROW),
    "parameter": lambda d: moss.quant_act_2level(torch.nn.Parameter(d["x"]), ROW),
    "small workspace": lambda d: moss.quant_act_2level(d["x"], ROW, workspace=torch.zeros(64, dtype=torch.uint8, device="cuda:0")),
    "maximum given": lambda d: moss.quant_act_2level_given_max(d["x"], d["x"].abs().max().view(1).view(torch.int16).int(), ROW | COL),
    "maximum of another type": lambda d: moss.quant_act_2level_given_max(d["x"], torch.ones(1, device="cuda:0"), ROW),
    "gemm": lambda d: (lambda q, w, s: moss.gemm_fp8_mx(q["q_row"], q["e_row"], q["s"], w, None, s))(*quantized(d)),
    "gemm into float32": lambda d: (lambda q, w, s: moss.gemm_fp8_mx(q["q_row"], q["e_row"], q["s"], w, None, s, out_dtype=torch.float32))(*quantized(d)),
    "gemm that accumulates": lambda d: (lambda q, w, s: moss.gemm_fp8_mx(q["q_row"], q["e_row"], q["s"], w, None, s, accumulate=True,
                                                                         out=torch.ones(64, 96, device="cuda:0")))(*quantized(d)),
    "gemm that accumulates BF16": lambda d: (lambda q, w, s: moss.gemm_fp8_mx(q["q_row"], q["e_row"], q["s"], w, None, s, accumulate=True))(*quantized(d)),
    "gemm into float16": lambda d: (lambda q, w, s: moss.gemm_fp8_mx(q["q_row"], q["e_row"], q["s"], w, None, s,
                                                                     out=torch.ones(64, 96, device="cuda:0").half()))(*quantized(d)),
    "gemm of two widths": lambda d: (lambda q, w, s: moss.gemm_fp8_mx(q["q_row"], q["e_row"], q["s"], w[:, :128].contiguous(), None, s))(*quantized(d)),
    "gemm of a view": lambda d: (lambda q, w, s: moss.gemm_fp8_mx(q["q_row"], q["e_row"], q["s"], w[:, ::2], None, s))(*quantized(d)),
    "swiglu": lambda d: moss.swiglu_bf16(d["x"], d["y"]),
    "swiglu strided": lambda d: moss.swiglu_bf16(d["wide"], d["wide"]),
    "swiglu of two strides": lambda d: moss.swiglu_bf16(d["wide"], d["y"]),
    "swiglu backward": lambda d: moss.swiglu_bf16_backward(d["x"], d["y"], d["y"]),
    "swiglu backward, outputs given": lambda d: moss.swiglu_bf16_backward(d["x"], d["y"], d["y"], torch.zeros_like(d["x"]), torch.zeros_like(d["x"]),
                                                                          torch.zeros(1, dtype=torch.int32, device="cuda:0"),
                                                                          torch.zeros(1, dtype=torch.int32, device="cuda:0")),
    "norm": lambda d: moss.add_rmsnorm_bf16(d["x"], d["gamma"], 1e-5),
    "norm with residual": lambda d: moss.add_rmsnorm_bf16(d["x"], d["gamma"], 1e-5, delta=d["y"]),
    "norm, whole eps": lambda d: moss.add_rmsnorm_bf16(d["x"], d["gamma"], 1),
    "norm, negative eps": lambda d: moss.add_rmsnorm_bf16(d["x"], d["gamma"], -1.0),
    "norm, narrow gamma": lambda d: moss.add_rmsnorm_bf16(d["x"], d["gamma"][:128], 1e-5),
    "norm backward": lambda d: moss.rmsnorm_bf16_backward(d["x"], d["gamma"], d["y"], 1e-5, d_res=d["x"]),
    "norm backward, float32": lambda d: moss.rmsnorm_bf16_backward(d["x"], d["gamma"], d["y"].float(), 1e-5),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CALLS))
def test_native_and_python_calls_agree(monkeypatch, data, name):
    native, python = both(monkeypatch, lambda: CALLS[name](data))
    torch.cuda.synchronize()
    same(native, python)


@pytest.mark.gpu
@pytest.mark.parametrize("bf16,transpose", [(False, True), (True, False)])
@pytest.mark.parametrize("wrong", [None, "step", "dtype", "args"])
def test_native_and_python_weight_steps_agree(monkeypatch, data, bf16, transpose, wrong):
    def call():
        w, m, v = data["w"].clone(), torch.zeros_like(data["w"]), torch.zeros_like(data["w"])
        state = moss.new_wscale_state(w.device)
        moss.weight_autoscale_init(w, state)
        g = data["g"].bfloat16() if bf16 else data["g"]
        args = adamw(0 if wrong == "step" else 1)
        out = moss.weight_autoscale_cast(w, m if wrong != "dtype" else m.double(), v, g, None if wrong == "args" else args, state, want_transpose=transpose)
        return out, w, m, v, state
    native, python = both(monkeypatch, call)
    torch.cuda.synchronize()
    same(native, python)


@pytest.mark.gpu
def test_native_calls_run_on_the_current_stream_and_leave_modes_to_python(monkeypatch, data):
    from torch.overrides import TorchFunctionMode

    class Count(TorchFunctionMode):
        n = 0

        def __torch_function__(self, func, types, args=(), kwargs=None):
            Count.n += func is torch.empty
            return func(*args, **(kwargs or {}))

    want = moss.quant_act_2level(data["x"], ROW)
    with Count():
        got = moss.quant_act_2level(data["x"], ROW)
    assert Count.n == 4                                  # q_row, e_row, s and the workspace
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        x = data["x"] * 1
        aside = moss.quant_act_2level(x, ROW)
    side.synchronize()
    torch.cuda.synchronize()
    same(want, got)
    same(want, aside)
