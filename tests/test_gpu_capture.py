"""Applies captured in a HIP graph as the first launch of their kernels in a process: nothing but kernels may be needed
then.  The graph is replayed with eager work in between and every replay is compared with the eager result."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import sys
import torch
import synthetic_inputs as si
from paper_2112_14640_amd import dirac

op, prec, nv = sys.argv[1], sys.argv[2], int(sys.argv[3])
dev = "cuda:0"
dtype = torch.complex128 if prec == "fp64" else torch.complex64
gen = torch.Generator(device=dev).manual_seed(5)
gauge = si.haar_su_n_t(gen, (12, 9, 8, 10, 4), 3, dev, dtype)
if op == "brillouin":
    gauge = dirac.brillouin_links(gauge)

def vector():
    u = si.complex_gaussian_t(gen, (12, 9, 8, 10, 3, 4, nv), dev, dtype)
    return torch.view_as_real(u).to(torch.bfloat16).contiguous() if prec == "bf16" else u

u, out = vector(), torch.empty_like(vector())
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):
    dirac.apply(op, gauge, u, 0.1, out=out)
for _ in range(4):
    u.copy_(vector())
    out.zero_()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, dirac.apply(op, gauge, u, 0.1))
print("captured", op, prec, nv)
"""


@pytest.mark.parametrize("op,prec,nv", [("brillouin", "fp64", 4), ("brillouin", "fp32", 4), ("brillouin", "bf16", 12),
                                        ("wilson", "fp32", 12)])
def test_first_launch_can_be_captured(op, prec, nv):
    r = subprocess.run([sys.executable, "-c", PROGRAM, op, prec, str(nv)], cwd=ROOT, capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and "captured" in r.stdout, r.stderr[-2000:]
