"""The binding on a torch build without the functions that it takes the raw
stream handle from: it imports, host calls work, and the stream comes from
torch's public interface."""
import subprocess
import sys

from conftest import ROOT

CODE = r"""
import types
import torch
for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
    if hasattr(torch._C, name):
        delattr(torch._C, name)
from paper_2609_36959_amd import binding as B
table, owner, plan, obj, feasible = B.cobalt_plan_layout(
    1, 2, 4, 3, torch.ones(4, 4), torch.ones(4))
assert sorted(set(table.ravel().tolist()) - {-1}) == [0, 1, 2, 3] and len(owner) == 4
torch.cuda.is_initialized = lambda: True
torch.cuda.current_stream = lambda: types.SimpleNamespace(cuda_stream=77)
assert B._stream(None) == 77
assert B._stream(types.SimpleNamespace(cuda_stream=5)) == 5
"""


def test_import_without_private_functions():
    r = subprocess.run([sys.executable, "-c", CODE], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
