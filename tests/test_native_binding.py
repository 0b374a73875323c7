"""The eager calls of the Linear in native code (csrc/ams_binding.cpp) against the same calls in Python: results, the stream they
go to, and everything that is not a plain tensor or an int or that is wrong, which takes the long way and raises there."""

import ctypes
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

import paper_2510_16045_amd as ams

torch = pytest.importorskip("torch")


def native(*a):
    from paper_2510_16045_amd import _binding

    return _binding.linear(*a)


def long_way(monkeypatch):
    monkeypatch.setattr(ams, "_call", lambda *a: None)


def test_what_is_not_on_the_gpu_or_no_tensor_is_left_alone():
    u8, f16 = torch.zeros(ams.ams_packed_bytes(ams.FP425, 16, 128), dtype=torch.uint8), torch.zeros(16, dtype=torch.float16)
    x, y = torch.zeros((2, 128), dtype=torch.float16), torch.zeros((2, 16), dtype=torch.float16)
    for entry in range(4):
        assert native(entry, u8, f16, x, 16, ams.FP425, y, 128) is None
        assert native(entry, None, f16, x, 16, ams.FP425, y, None) is None
        assert native(entry, u8, f16, x, 16.0, ams.FP425, y, None) is None
    assert native() is None and native(0, u8) is None and native("0", u8, f16, x, 16, ams.FP425, y, None) is None
    with pytest.raises(ValueError):
        ams.ams_linear(u8, f16, x, 16, ams.FP425, out=y)


def in_a_copy(tmp_path, code, spoil=None):
    """Runs code in a process of its own with a copy of the built package, from which `spoil` may take or change something."""
    package = tmp_path / "paper_2510_16045_amd"
    shutil.copytree(os.path.dirname(ams.__file__), package, ignore=shutil.ignore_patterns("__pycache__"))
    if spoil:
        spoil(package)
    run = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env={**os.environ, "PYTHONPATH": str(tmp_path)}, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr
    return run.stdout


def test_a_copy_of_the_package_calls_its_own_library(tmp_path):
    code = """
import paper_2510_16045_amd as ams
ams._bind_call()
from paper_2510_16045_amd import _binding
assert ams._call is _binding.linear
print(*sorted({line.split()[-1] for line in open("/proc/self/maps") if "libams" in line}))
"""
    assert in_a_copy(tmp_path, code).split() == [str(tmp_path / "paper_2510_16045_amd" / "libams.so")]


BIND_TWICE = """
import warnings
import paper_2510_16045_amd as ams
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    ams._call()
    ams._call()
print(len(seen), *{w.category.__name__ for w in seen}, ams._call(), *{str(w.message) for w in seen})
"""


def native_files(package):
    return [f for f in package.iterdir() if f.name.startswith("_binding.") and f.suffix == ".so"]


def test_a_binding_that_does_not_load_is_said_once(tmp_path):
    def spoil(package):
        for f in native_files(package):
            f.write_bytes(b"no library")

    assert in_a_copy(tmp_path, BIND_TWICE, spoil).startswith("1 RuntimeWarning None ")


def test_a_binding_for_another_torch_is_declined(tmp_path):
    other = "import torch; torch.version.git_version = 'f' * 40" + BIND_TWICE
    assert in_a_copy(tmp_path, other).startswith("1 RuntimeWarning None ")


def test_a_package_without_the_binding_is_whole(tmp_path):
    assert in_a_copy(tmp_path, BIND_TWICE, lambda package: [f.unlink() for f in native_files(package)]).split() == ["0", "None"]


def test_the_library_is_built_where_torch_has_no_headers(monkeypatch):
    import __graft_entry__ as entry

    ran = []
    monkeypatch.setattr(entry, "_run", ran.append)
    monkeypatch.setitem(sys.modules, "torch.utils", None)
    entry.build()
    assert any(entry.LIB in cmd for cmd in ran) and not any("ams_binding" in word for cmd in ran for word in cmd)


def test_an_output_that_is_too_small_is_refused():
    W, scales, x = torch.zeros(ams.ams_packed_bytes(ams.FP425, 16, 128), dtype=torch.uint8), torch.zeros(16, dtype=torch.float16), torch.zeros((2, 128), dtype=torch.float16)
    small, small_w, w = torch.zeros(31, dtype=torch.float16), torch.zeros((15, 128), dtype=torch.float16), torch.zeros((16, 128), dtype=torch.float16)
    for call in (
        lambda: ams.ams_linear(W, scales, x, 16, ams.FP425, out=small), lambda: ams.ams_linear_ws(W, scales, x, 16, ams.FP425, None, out=small),
        lambda: ams.ams_linear_static_ws(W, scales, x, 16, ams.FP425, out=small), lambda: ams.ams_linear_grouped(W, scales, 128, x, 16, ams.FP425, out=small),
        lambda: ams.ams_fp16_linear(w, x, out=small), lambda: ams.ams_fp16_linear_ws(w, x, None, out=small),
        lambda: ams.ams_dequant(ams.FP425, W, scales, 16, 128, out=small_w), lambda: ams.ams_dequant_grouped(ams.FP425, W, scales, 128, 16, 128, out=small_w),
    ):
        with pytest.raises(ValueError, match="out must hold"):
            call()


def test_a_tensor_on_another_device_is_refused(monkeypatch):
    class There:
        is_cuda = True
        is_contiguous = lambda self: True
        get_device = lambda self: 1
        data_ptr = lambda self: 4096

    monkeypatch.setattr(ams, "_devices", 0)
    monkeypatch.setattr(torch.cuda, "device_count", lambda: 2)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 1)
    assert ams._dev_ptr(There()) == 4096
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    for _ in range(2):
        with pytest.raises(ValueError, match="current device"):
            ams._dev_ptr(There())


def test_a_daemon_thread_in_a_call_ends_with_the_interpreter(tmp_path):
    # the binding's own code around a library that takes 2 ms for a call: when the interpreter ends, the thread is in one
    (tmp_path / "in_call.cpp").write_text(f"""
#include "{os.path.dirname(ams.__file__)}/csrc/ams_binding.cpp"
#include <unistd.h>
static PyObject* run(PyObject*, PyObject*) {{
  lib.linear = [](const void*, const uint16_t*, const uint16_t*, uint16_t*, int, int64_t, int64_t, int, void*) {{ return usleep(2000), (int)AMS_OK; }};
  return PyLong_FromLong(call_unlocked(Call{{}}));
}}
static PyMethodDef only[] = {{{{"run", run, METH_NOARGS, nullptr}}, {{nullptr, nullptr, 0, nullptr}}}};
static PyModuleDef here = {{PyModuleDef_HEAD_INIT, "in_call", nullptr, -1, only, nullptr, nullptr, nullptr, nullptr}};
PyMODINIT_FUNC PyInit_in_call() {{ return PyModule_Create(&here); }}
""")
    import __graft_entry__ as g

    if g.binding_includes() is None:
        pytest.skip("no headers of torch: there is no native binding")
    subprocess.run(g.binding_command(g._hipcc(), g.binding_includes(), str(tmp_path / "in_call.cpp"), str(tmp_path / "in_call.so")), check=True, timeout=300)
    code = """
import threading, time, torch, in_call

class Last:  # gone when the interpreter has begun to end
    def __del__(self, sleep=time.sleep):
        sleep(0.1)

def calls():
    while True:
        assert in_call.run() == 0

last = Last()
threading.Thread(target=calls, daemon=True).start()
time.sleep(0.05)
"""
    end = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, timeout=300)
    assert (end.returncode, end.stderr) == (0, "")


@pytest.fixture
def problem():
    def make(M=3, N=300, K=520, fmt=ams.FP425, group=128):
        rng = np.random.default_rng(4)
        codes = (rng.integers(0, 32, size=(N, K), dtype=np.uint8) & 0xFE) | 1
        W = torch.from_numpy(ams.ams_pack_codes(fmt, codes)).cuda()
        gen = torch.Generator(device="cuda").manual_seed(5)
        X = torch.randn((M, K), generator=gen, device="cuda").half()
        run = torch.rand(ams.ams_group_scales_count(fmt, N, K, group), generator=gen, device="cuda").half()
        ws = torch.zeros(max(16, ams.ams_linear_workspace_bytes(fmt, M, N, K)), dtype=torch.uint8, device="cuda")
        scales = torch.rand(N, generator=gen, device="cuda").half()
        return W, scales, run, X, N, fmt, ws, group

    return make


def calls(p):
    W, scales, run, X, N, fmt, ws, group = p
    return {
        "plain": lambda out: ams.ams_linear(W, scales, X, N, fmt, out=out),
        "ws": lambda out: ams.ams_linear_ws(W, scales, X, N, fmt, ws, out=out),
        "no ws": lambda out: ams.ams_linear_ws(W, scales, X, N, fmt, None, out=out),
        "static": lambda out: ams.ams_linear_static_ws(W, scales, X, N, fmt, out=out),
        "grouped": lambda out: ams.ams_linear_grouped(W, run, group, X, N, fmt, out=out),
    }


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [dict(), dict(M=32, N=256, K=14336), dict(M=1, N=5, K=7), dict(M=8, N=4096, K=12808)])
def test_results_are_the_long_ways(monkeypatch, problem, shape):
    p = problem(**shape)
    M, N = p[3].shape[0], p[4]
    got = {}
    for name, call in calls(p).items():
        out = torch.full((M, N), 9.0, dtype=torch.float16, device="cuda")
        assert call(out) is out
        got[name] = out
    assert native(0, p[0], p[1], p[3], p[4], p[5], got["plain"], None) is got["plain"]  # the native way is the one taken
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        on_side = calls(p)["plain"](torch.empty_like(got["plain"]))
    side.synchronize()
    graph, captured = torch.cuda.CUDAGraph(), torch.zeros_like(got["plain"])
    with torch.cuda.graph(graph):
        calls(p)["plain"](captured)
    for _ in range(3):
        captured.zero_()
        graph.replay()
        assert torch.equal(captured, got["plain"])
    long_way(monkeypatch)
    for name, call in calls(p).items():
        assert torch.equal(call(torch.empty_like(got[name])), got[name]), name
        assert torch.equal(call(None), got[name]), name
    assert torch.equal(on_side, got["plain"])


@pytest.mark.gpu
def test_what_is_wrong_raises_as_before(monkeypatch, problem):
    W, scales, run, X, N, fmt, ws, group = problem()
    out = torch.empty((X.shape[0], N), dtype=torch.float16, device="cuda")
    wrong = [
        (W[:-1], scales, X, N, fmt, out), (W.view(torch.int8), scales, X, N, fmt, out), (W, scales[:-1], X, N, fmt, out), (W, scales.float(), X, N, fmt, out),
        (W, scales, X.float(), N, fmt, out), (W, scales, X.t().contiguous().t(), N, fmt, out), (W, scales, X[0], N, fmt, out), (W, scales, X.cpu(), N, fmt, out),
        (W, scales, X, float(N), fmt, out), (W, scales, X, N, 99, out), (W, scales, X, -N, fmt, out), (W, scales, X, N, fmt, out.t()), (W, scales, X, N, fmt, out.float()),
        (W, scales, X.repeat(20, 1), N, fmt, out), (W, scales, X, 1 << 70, fmt, out), (None, scales, X, N, fmt, out), (W, scales, X, N, fmt, "out"),
        (W, scales, X, N, fmt, out[:-1]), (W, scales, X, N, fmt, out.flatten()[:-1]),
    ]

    def outcome(args):
        try:
            ams.ams_linear(*args[:5], out=args[5])
        except (Exception, ctypes.ArgumentError) as e:
            return type(e), str(e)
        return None

    assert native(0, W, scales, X, N, fmt, out[:-1], None) is None
    first = [outcome(a) for a in wrong]
    assert all(first), first
    larger = torch.full((X.shape[0] + 1, N), 9.0, dtype=torch.float16, device="cuda")  # a buffer for a larger batch
    assert ams.ams_linear(W, scales, X, N, fmt, out=larger) is larger
    assert torch.equal(larger[:-1], ams.ams_linear(W, scales, X, N, fmt)) and (larger[-1] == 9.0).all()
    long_way(monkeypatch)
    assert [outcome(a) for a in wrong] == first


@pytest.mark.gpu
def test_other_tensors_take_the_long_way(problem):
    W, scales, run, X, N, fmt, ws, group = problem()
    out = torch.empty((X.shape[0], N), dtype=torch.float16, device="cuda")

    class Sub(torch.Tensor):
        pass

    assert native(0, W, scales, X.as_subclass(Sub), N, fmt, out, None) is None
    assert torch.equal(ams.ams_linear(W, scales, X.as_subclass(Sub), N, fmt, out=out), ams.ams_linear(W, scales, X, N, fmt))
    assert native(0, W, torch.nn.Parameter(scales), X, N, fmt, out, None) is out
    seen = []

    def wrapped(x):
        seen.append(native(0, W, scales, x, N, fmt, out, None))
        return x

    torch.vmap(wrapped)(X.expand(2, *X.shape).contiguous())
    torch.func.jvp(wrapped, (X,), (X,))
    assert seen == [None, None]
