"""tune[1], the FP32 row form, is taken where it is set, also in rows that the default
gives the widest kernel (more than 20 markers a lane): the capacity the library reports
is that of the form asked for, and the results are those of the default."""
import os
import re
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu

CODE = """
import sys
sys.path.insert(0, {root!r})
import torch
from paper_1804_03901_amd import avl, inputs
w = inputs.bump_on_tail(nx=128, nv=12, ppc=24, seed=7)
m = inputs.markers(w)
ref = None
for form in (0, 1, 2):
    sim = avl.Simulation(w, m[0], m[1].reshape(-1), m[2], precision=avl.AVL_FP32, tune={{avl.TUNE_RECON_FORM: form}})
    out = sim.reconstruct(want_D=True)
    ref = ref or out
    assert all(torch.equal(a, b) for a, b in zip(out, ref))
    sim.close()
print("done")
"""


def test_row_form_is_taken_in_long_rows():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = subprocess.run([sys.executable, "-c", CODE.format(root=ROOT)], capture_output=True, text=True, timeout=110,
                       env=dict(os.environ, AVL_DEBUG="1"))
    assert r.returncode == 0 and r.stdout.strip().endswith("done"), r.stderr[-2000:]
    caps = [int(c) for c in re.findall(r"recon cap (\d+)", r.stderr)]
    assert caps == [64 * 29, 64 * 21, 64 * 21]
