"""What needs the native binding and what does not, without a GPU."""
import subprocess
import sys

from tests.conftest import ROOT


def test_library_without_the_binding():
    """_binding.so is built for one Python and one torch. Where it cannot be
    imported, the library loads and the calls that need only the library work;
    the others say what is missing."""
    code = """
import sys
sys.modules["paper_2207_10284_amd._binding"] = None          # its import raises ImportError
import torch
from paper_2207_10284_amd import ops
lib = ops.load()
assert ops.forward_workspace_bytes(1, 1, 64, 64, 1) > 0
assert lib.mra_last_hip_error() == 0
try:
    ops.pool(torch.zeros(1, 1, 32, 32))
except ValueError as e:
    assert "ROCm device" in str(e)
else:
    raise SystemExit("a CPU tensor was accepted")
q = torch.zeros(1, 1, 32, 32)
for call in (ops.attention_forward, ops.sparse_attention_forward, ops.attention_forward_global, ops.mra_attention):
    try:
        call(q, q, q, 1)
    except RuntimeError as e:
        assert "binding is not built" in str(e), e
    else:
        raise SystemExit(f"{call} ran without the binding")
print("fine")
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip().endswith("fine"), r.stdout + r.stderr
