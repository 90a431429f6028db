"""The first solve of a process: a resident handle takes no more device memory in it than
one that launches per sweep (whose first solve loads code).  The queue that the first
cooperative launch creates, and its kernels' scratch memory, belong to the setup, so that
vtm_solve_noalloc keeps its promise from the first call on.
"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import sys
import torch
import paper_0910_0663_amd as vtm
import workloads
w = workloads.make(1)
b = torch.as_tensor(w.b, device="cuda")
x = torch.empty_like(b)
s = vtm.Solver(w.A, w.part, w.Z, timing=int(sys.argv[1]))
torch.cuda.synchronize()
free = torch.cuda.mem_get_info()[0]
s.solve(b, 1e-10, x)
torch.cuda.synchronize()
print("taken", free - torch.cuda.mem_get_info()[0])
"""


def taken(timing):
    out = subprocess.run([sys.executable, "-c", CHILD, str(timing)], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr[-2000:]
    return int(out.stdout.split()[-1])


def test_first_solve_takes_no_memory_for_a_cooperative_launch():
    assert taken(0) <= taken(1)
