"""csrc/call.cpp on the CPU: the same source built for host tensors, with its allocations and the wrapping of its results
watched, against a library that only counts its calls."""
import ctypes
import importlib.util
import os
import subprocess

import pytest
import torch

from paper_2502_08141_amd import build

_WATCH = """
extern "C" { int watch_empties, watch_held, watch_fail; }
static at::Tensor watched_empty(at::IntArrayRef sizes, const at::TensorOptions& o) {
    ++watch_empties; watch_held += PyGILState_Check();
    return at::empty(sizes, o);
}
static PyObject* watched_wrap(at::Tensor t) {
    if (watch_fail == 1) throw std::bad_alloc();
    if (watch_fail == 2) { PyErr_NoMemory(); return nullptr; }
    return THPVariable_Wrap(std::move(t));
}
"""
N, K, C, M, R = 8, 128, 3, 5, 4


@pytest.fixture(scope="module")
def native(tmp_path_factory):
    d = tmp_path_factory.mktemp("call")
    text = open(os.path.join(build.CSRC, "call.cpp")).read()
    for old, new, least in (("t.is_cuda()", "t.is_cpu()", 1), ("(void*)c10::hip::getCurrentHIPStream().stream()", "nullptr", 1),
                            ("at::empty(", "watched_empty(", 1), ("THPVariable_Wrap(", "watched_wrap(", 5)):
        assert text.count(old) >= least
        text = text.replace(old, new)
    text = text.replace("namespace {\n", _WATCH + "namespace {\n", 1)
    (d / "call.cpp").write_text(text)
    so = str(d / "_lowra_call.so")
    subprocess.run([a if a != "-O2" else "-O0" for a in build.call_command(str(d / "call.cpp"), so)], check=True)
    spec = importlib.util.spec_from_file_location("_lowra_call", so)
    call = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(call)

    vp, i, f, n = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_size_t
    lib = type("lib", (), {"calls": 0, "status": 0, "keep": []})

    def entry(*types):
        def count(*_):
            lib.calls += 1
            return lib.status
        lib.keep.append(ctypes.CFUNCTYPE(i, *types)(count))
        return ctypes.cast(lib.keep[-1], vp).value

    call.init(*[entry(vp, vp, vp, vp, vp, i, vp, vp, i, f, vp, vp, n, vp) for _ in range(2)], entry(vp, i, i, i, vp),
              entry(vp, vp, vp, i, vp, vp, i, f, vp, vp, vp, n, vp), entry(vp, vp, vp, i, i, vp, vp, vp, vp, vp, n, vp),
              entry(vp, vp, vp, vp, i, vp, vp))
    watch = {k: ctypes.c_int.in_dll(ctypes.CDLL(so), "watch_" + k) for k in ("empties", "held", "fail")}
    return call, lib, watch


def _calls(call):
    z = lambda *s, dtype=torch.bfloat16: torch.zeros(s, dtype=dtype)
    state = ((4096, N, K, C, 100, False), z(100, dtype=torch.uint8), z(N, K // 64, dtype=torch.float32), z(C, 16, dtype=torch.float32))
    x, dY, A, B, side, ws = z(M, K), z(M, N), z(R, K), z(N, R), z(M, 64), z(512, dtype=torch.uint8)
    return {"fwd": (lambda: call.linear(0, *state, x, A, B, 1.0, ws), [(M, N)]),
            "bwd": (lambda: call.linear(1, *state, dY, None, None, 1.0, ws), [(M, K)]),
            "grads": (lambda: call.grads(state[0], x, dY, A, B, 1.0, ws), [(R, K), (N, R)]),
            "grads_from_side": (lambda: call.grads_from_side(state[0], x, dY, R, side, side, ws), [(R, K), (N, R)]),
            "dequantize": (lambda: call.dequantize(*state), [(N, K)])}


@pytest.mark.parametrize("which", ["fwd", "bwd", "grads", "grads_from_side", "dequantize"])
def test_allocations_and_failures(native, which):
    call, lib, watch = native
    run, shapes = _calls(call)[which]
    lib.calls, lib.status = 0, 0
    for v in watch.values():
        v.value = 0
    res = run()
    assert [tuple(t.shape) for t in (res if isinstance(res, tuple) else (res,))] == shapes and lib.calls == 1
    # other threads run while an output is allocated
    assert watch["empties"].value == len(shapes) and watch["held"].value == 0
    # "nothing launched" is what None says
    for watch["fail"].value in (1, 2):
        assert run() is None and lib.calls == 1
    watch["fail"].value = 0
    lib.status = 4
    assert run() == 4 and lib.calls == 2
