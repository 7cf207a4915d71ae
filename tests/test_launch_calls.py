"""The launch calls of the Python binding (csrc/py_launch.cpp, and ctypes where that is not built): what they take as
tensors, plans and streams, on a group without rows, which launches nothing."""
import ctypes as C
import os
import subprocess
import sys
import sysconfig
from collections import deque

import pytest

from paper_1911_11576_amd import BoundArgs, FsError, Plan, binding, build
from workloads import graphs


class Tensor:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        return self.address


@pytest.fixture(scope="module", autouse=True, params=["native", "ctypes"])
def calls(request):
    binding.lib()
    kept = binding._native
    if request.param == "ctypes":
        binding._native = binding._CtypesCalls()
    elif isinstance(kept, binding._CtypesCalls):
        pytest.skip("_launch is not built for this interpreter")
    yield
    binding._native = kept


@pytest.fixture(scope="module")
def plan(calls):
    with Plan(graphs.layernorm_fwd(0, 768, "f32", 1e-5)) as p:
        yield p


TENSORS = [[4096, 8192, 16384], (Tensor(4096), 8192, Tensor(16384)), deque([Tensor(4096)] * 3), range(4096, 4096 * 4, 4096)]


@pytest.mark.parametrize("ins", TENSORS, ids=lambda t: type(t).__name__)
@pytest.mark.parametrize("stream", [0, C.c_void_p(0), C.c_void_p(64)], ids=["int", "null", "c_void_p"])
def test_accepted(plan, ins, stream):
    plan.launch(ins, [32768], stream)
    binding.fs_launch(plan._h, ins, (Tensor(32768),), stream)
    binding.fs_launch(C.c_void_p(plan._h), ins, [32768], stream)
    plan.launch_static(ins, [32768], stream)
    plan.launch_bound(BoundArgs(ins, [32768]), stream)
    plan.launch_bound(BoundArgs(ins, [32768]), None)


@pytest.mark.parametrize("ins, outs, error", [
    ([4096, 8192], [32768], FsError),                    # counts
    ([4096, 8196, 16384], [32768], FsError),             # alignment of gamma, which has elements
    ([4096] * 100, [32768], FsError),                    # more than the local array holds
    ([4096, 8192, -1], [32768], OverflowError),
    ([4096, 8192, 1 << 64], [32768], OverflowError),
    ([4096, 8192, 1.5], [32768], AttributeError),
    ([4096, 8192, Tensor(1.5)], [32768], TypeError),
    ([4096, 8192, None], [32768], AttributeError),
    (iter([4096, 8192, 16384]), [32768], TypeError),     # no length
    (None, [32768], TypeError),
])
def test_refused(plan, ins, outs, error):
    with pytest.raises(error):
        plan.launch(ins, outs, 0)
    with pytest.raises(error):
        plan.launch_static(ins, outs, 0)


class Stream:
    """What a torch.cuda.Stream is to ctypes."""
    _as_parameter_ = C.c_void_p(64)


@pytest.mark.parametrize("stream", [Stream(), C.byref(C.c_uint64()), (C.c_uint64 * 4)(), C.pointer(C.c_uint64())], ids=lambda s: type(s).__name__)
def test_streams_that_ctypes_takes(plan, stream):
    plan.launch([4096, 8192, 16384], [32768], stream)
    plan.launch_static([4096, 8192, 16384], [32768], stream)
    plan.launch_bound(BoundArgs([4096, 8192, 16384], [32768]), stream)


@pytest.mark.parametrize("stream", [C.c_int(3), 1.5, [], Tensor(64)], ids=lambda s: type(s).__name__)
def test_streams_that_ctypes_refuses(plan, stream):
    for call in (lambda: plan.launch([4096, 8192, 16384], [32768], stream), lambda: plan.launch_static([4096, 8192, 16384], [32768], stream),
                 lambda: plan.launch_bound(BoundArgs([4096, 8192, 16384], [32768]), stream)):
        with pytest.raises(C.ArgumentError):
            call()


def test_a_list_that_shrinks_while_it_is_read(plan):
    class Shrinks(Tensor):
        def data_ptr(self):
            ins.clear()
            return self.address
    ins = [4096, Shrinks(8192), 16384]
    with pytest.raises((RuntimeError, IndexError)):
        plan.launch(ins, [32768], 0)


def test_a_closed_plan_is_refused():
    p = Plan(graphs.layernorm_fwd(0, 768, "f32", 1e-5))
    p.close()
    for call in (lambda: p.launch([4096] * 3, [32768], 0), lambda: p.launch_bound(BoundArgs([4096] * 3, [32768]), 0)):
        with pytest.raises(FsError):
            call()


def test_an_interpreter_that_launch_was_not_built_for():
    code = ("import sys; sys.modules['paper_1911_11576_amd._launch'] = None\n"
            "from paper_1911_11576_amd import Plan, binding\n"
            "from workloads import graphs\n"
            "with Plan(graphs.layernorm_fwd(0, 768, 'f32', 1e-5)) as p:\n"
            "    p.launch([4096] * 3, [32768], 0)\n"
            "assert isinstance(binding._native, binding._CtypesCalls)\n")
    subprocess.run([sys.executable, "-c", code], check=True, timeout=120, cwd=os.path.dirname(build.HERE))


def built(tmp_path, monkeypatch, environ):
    """What a build in this environment runs and writes, with the compiler left out."""
    commands = []
    monkeypatch.setattr(build, "OBJ", str(tmp_path / "obj"))
    monkeypatch.setattr(build, "PY_LIB", str(tmp_path / "_launch.so"))
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **_: commands.append(cmd) or subprocess.CompletedProcess(cmd, 0, "", ""))
    monkeypatch.delenv("FS_LIB_OUT", raising=False)
    for name, value in environ.items():
        monkeypatch.setenv(name, value)
    build.build()
    return [cmd[cmd.index("-o") + 1] for cmd in commands]


def test_a_library_built_elsewhere_leaves_the_package_alone(tmp_path, monkeypatch):
    assert str(tmp_path / "_launch.so") in built(tmp_path, monkeypatch, {})
    assert str(tmp_path / "_launch.so") not in built(tmp_path, monkeypatch, {"FS_LIB_OUT": str(tmp_path / "lib.so")})


def test_a_build_without_python_headers(tmp_path, monkeypatch):
    monkeypatch.setattr(sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    (tmp_path / "_launch.so").write_text("of an earlier build")
    assert str(tmp_path / "_launch.so") not in built(tmp_path, monkeypatch, {}) and not (tmp_path / "_launch.so").exists()
