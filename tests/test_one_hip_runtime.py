"""One HIP runtime in a process that calls the binding before it has imported
torch (host only, in processes of their own): libttm.so names its runtime by
version and torch brings its own, so the library comes after torch.  With two of
them, device memory of the one is none of the other's."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FIRST_CALLS = {
    "lib": "T.lib()",
    # refused for want of a GPU, behind whatever the call loads first
    "multiply_vjp": """
ones = [np.ones((1, 2, 1)), np.ones((1, 2, 1))]
try:
    T.multiply_vjp(ones, ones, 1, 0.0, ones)
except Exception:
    pass
""",
}


@pytest.mark.parametrize("call", sorted(FIRST_CALLS))
def test_library_comes_after_torch(call):
    code = """
import sys
import numpy as np
import paper_2410_19747_amd as T
assert "torch" not in sys.modules
%s
import torch
T.lib()
print("\\n".join(sorted({l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l})))
""" % FIRST_CALLS[call]
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, HIP_VISIBLE_DEVICES=""))
    assert p.returncode == 0, p.stderr[-2000:]
    assert len(p.stdout.split()) == 1, p.stdout
