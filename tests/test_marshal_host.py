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
