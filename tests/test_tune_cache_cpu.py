"""Shapes in a file named by PSS_TUNE_CACHE belong to the kernels that they were
timed for: entries under the signature of earlier kernels are read and not
applied, entries under today's are."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SIZE = """
import numpy as np, torch, ctypes
from paper_2207_00426_amd import pss
b = pss.Batch(pss.MODEL_LINEAR, torch.float64, 4, 2, np.array([0, 900, 3000]), np.zeros(4),
              np.eye(4), device="cpu")
g = b.gamma_from_numpy(dict(F=np.eye(4), c=np.zeros(4), SL=np.eye(4), H=np.eye(4)[:2],
                            d=np.zeros(2), SO=np.eye(2)))
y, (m, N) = torch.zeros(2, 3000, dtype=torch.float64), b.prior_nominal()
print(pss.batched_workspace_size([(b, y, m, N, g)]))
"""


def _size(path=None):
    env = dict(os.environ)
    env.pop("PSS_TUNE_CACHE", None)
    if path:
        env["PSS_TUNE_CACHE"] = str(path)
    return int(subprocess.run([sys.executable, "-c", SIZE], cwd=ROOT, env=env, check=True,
                              stdout=subprocess.PIPE, text=True).stdout)


def test_only_entries_for_these_kernels_are_applied(tmp_path):
    plain = _size()
    old, new = tmp_path / "old.txt", tmp_path / "new.txt"
    old.write_text('"f64|0:4:B2:L12" 256 1 1\n')
    new.write_text('"v2|f64|0:4:B2:L12:N12:g0" 256 1 1\n')
    assert _size(old) == plain
    assert _size(new) != plain
