"""The native marshalling (csrc/marshal.cpp) on a host without a GPU: whatever it cannot take is left to the Python path, which
raises.  Each call runs in a process of its own: a C++ exception that leaves a C function ends the process."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = """
import torch
import paper_2508_00960_amd as ph
prob = ph.make_problem(256, 4, 8, 32)
step = ph.make_problem(256, 4, 8, 32, layers=2)
sparse = torch.sparse_coo_tensor(torch.zeros(1, 1, dtype=torch.long), torch.ones(1), (4,))
two = [None, None]
"""


def run(code):
    env = {**os.environ, "HIP_VISIBLE_DEVICES": "", "PYTHONPATH": ROOT}
    return subprocess.run([sys.executable, "-c", HEAD + code], capture_output=True, text=True, env=env, cwd=ROOT, timeout=300)


@pytest.mark.parametrize("call,raises", [
    # no stream to ask for without a device: the argument errors come all the same
    ("ph.layer_fwd(prob, None, None, None, None, None, None, None, None, None)", "X is NULL"),
    ("ph.layer_bwd(prob, *[None] * 14)", "dY is NULL"),
    ("ph.ffn_step(step, None, None, two, two, two, two, mode='forward')", "X0 is NULL"),
    # tensors whose queries throw
    ("ph.layer_fwd(prob, None, None, None, None, None, None, None, None, None, workspace=sparse)", "RuntimeError"),
    ("ph.ffn_step(step, None, None, two, two, two, two, mode='forward', workspace=sparse)", "RuntimeError"),
    # arguments that are no numbers
    ("ph.ffn_step(step, None, None, two, two, two, two, lr='much')", "ValueError"),
])
def test_exceptions_reach_python(call, raises):
    out = run(call)
    assert out.returncode == 1 and raises in out.stderr, (out.returncode, out.stderr[-2000:])


def copy_of_package(tmp_path):
    import shutil
    shutil.copytree(os.path.join(ROOT, "paper_2508_00960_amd"), tmp_path / "paper_2508_00960_amd")
    shutil.copytree(os.path.join(ROOT, "include"), tmp_path / "include")
    return tmp_path / "paper_2508_00960_amd" / "_marshal.so"


def run_copy(tmp_path, code, path):
    env = {**os.environ, "HIP_VISIBLE_DEVICES": "", "PYTHONPATH": str(tmp_path), "PATH": path}
    return subprocess.run([sys.executable, "-c", HEAD + code], capture_output=True, text=True, env=env, cwd=tmp_path, timeout=300)


NULL_X = "ph.layer_fwd(prob, None, None, None, None, None, None, None, None, None)"


def test_package_works_without_the_native_module(tmp_path):
    """No module and no compiler to build it with."""
    copy_of_package(tmp_path).unlink()
    out = run_copy(tmp_path, "assert ph.workspace_bytes(prob) > 0\n" + NULL_X, path=str(tmp_path))
    assert out.returncode == 1 and "X is NULL" in out.stderr and "marshalled in Python" in out.stderr, out.stderr[-2000:]


@pytest.mark.parametrize("compiler", [True, False])
def test_stale_native_module_is_not_used(tmp_path, compiler):
    """Built from another header, for instance: rebuilt where that can be done, else left alone."""
    so = copy_of_package(tmp_path)
    with open(tmp_path / "include" / "phantom.h", "a") as f:
        f.write("/* changed */\n")
    code = "ph.load()\nfrom paper_2508_00960_amd import binding, build\nprint(binding._fast.__name__, build.marshal_is_current())\n" + NULL_X
    out = run_copy(tmp_path, code, path=os.environ["PATH"] if compiler else str(tmp_path))
    want = "paper_2508_00960_amd._marshal True" if compiler else "_PythonOnly False"
    assert out.returncode == 1 and "X is NULL" in out.stderr and out.stdout.strip() == want, (out.stdout, out.stderr[-2000:])


def test_load_is_never_half_done():
    """At no bytecode of load() may another thread see the library and not the marshalling that calls go through."""
    out = run("""
import sys
from paper_2508_00960_amd import binding
seen = 0
def trace(frame, event, arg):
    global seen
    if frame.f_code.co_filename != binding.__file__:
        return None
    frame.f_trace_opcodes = True
    seen += event == "opcode"
    assert binding._lib is None or binding._fast is not None
    return trace
sys.settrace(trace)
binding.load()
sys.settrace(None)
assert seen > 100 and binding._lib is not None
print("whole")
""")
    assert out.returncode == 0 and out.stdout.strip() == "whole", out.stderr[-2000:]


def test_threads_load_together():
    out = run("""
import threading
gate, errors = threading.Barrier(8), []
def call():
    gate.wait()
    try:
        """ + NULL_X + """
    except ph.PhantomError:
        return
    errors.append("no error")
threads = [threading.Thread(target=call) for _ in range(8)]
for t in threads: t.start()
for t in threads: t.join()
print(errors)
""")
    assert out.returncode == 0 and out.stdout.strip() == "[]" and "Traceback" not in out.stderr, out.stderr[-2000:]
