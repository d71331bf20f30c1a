"""The allocation-free apply when nothing of the plane kernels has run in the
process: its first call on a GPU loads every kernel the apply may launch, so
that a later first launch under a stream capture loads no code object there.

A fresh process: the first call is on an empty plan (it launches nothing), the
second, under a capture, launches the plane kernels for the first time.  The
graph is replayed three times, with eager work between the replays, and each
replay gives the bits of the eager apply."""
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_SCRIPT = r"""
import sys
import numpy as np
import torch
sys.path.insert(0, sys.argv[1])
import paper_1401_7441_amd as W
from tests.test_gpu_parity import _sphere_case
dtype = getattr(torch, sys.argv[2])
case = _sphere_case(nsf=3, seed_shift=21)
stream = torch.cuda.Stream()
with torch.cuda.stream(stream):
    ctx = W.Context(case.g.h, case.g.grid_n)
    empty = W.Plan(ctx, case.rec[:0], case.segs[:0])
    plan = W.Plan(ctx, case.rec, case.segs)
    assert plan.workspace_bytes(W.F64) <= W.STATIC_WORKSPACE_BYTES
    psi = torch.tensor(case.psi, dtype=dtype, device="cuda")
    pot = torch.tensor(case.pot, dtype=dtype, device="cuda")
    out = torch.zeros(plan.info["out_coefs"], dtype=dtype, device="cuda")
    ek = torch.zeros(3, dtype=torch.float64, device="cuda")
    ep = torch.zeros_like(ek)
    W.apply_local_ham_static(empty, psi, pot, out)
    torch.cuda.synchronize()
    print("capture", flush=True)
    g = torch.cuda.CUDAGraph()
    g.capture_begin()
    W.apply_local_ham_static(plan, psi, pot, out, ek, ep)
    g.capture_end()
    got = []
    for rep in range(3):
        out.zero_(), ek.zero_(), ep.zero_()
        g.replay()
        torch.cuda.synchronize()
        got.append([t.cpu().numpy().copy() for t in (out, ek, ep)])
    print("eager", flush=True)
    W.apply_local_ham(plan, psi, pot, out, ek, ep)
    torch.cuda.synchronize()
    for rep in range(3):
        for a, t in zip(got[rep], (out, ek, ep)):
            assert np.any(a) and np.array_equal(a, t.cpu().numpy()), rep
print("ok", flush=True)
"""


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_plane_kernels_first_launched_under_a_capture(dtype):
    print(f"case: static apply, first launch under a capture, {dtype}", flush=True)
    r = subprocess.run([sys.executable, "-c", _SCRIPT, ROOT, dtype], cwd=ROOT,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
    assert r.stdout.rstrip().endswith("ok")
