"""Graphs destroyed right after a launch, without waiting for it: plans of one and
of several bins, and of several chunks per bin.  A graph is linear, also over bins;
the launches run to their end with the bits of the eager apply."""
import numpy as np
import pytest

from tests.test_gpu_batching import _buffers, _mixed_case
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W


@pytest.fixture(scope="module")
def many():
    """150 functions of 7 to 21 points per axis: two LDS sizes of the back pass
    with 64 functions or more on either side."""
    base = _mixed_case(nsf=10, seed=5)
    lrs = [base.lrs[k % 10] for k in range(150)]
    g = base.g
    g.centers = np.repeat(g.centers, 15, axis=0)
    g.envelope_sigma = np.tile(g.envelope_sigma, 15)
    return Case(g, lrs)


@pytest.mark.parametrize("nbins", [1, 3, 6])
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_destroy_right_after_launch(many, nbins, dtype):
    dt = getattr(torch, dtype)
    plan = W.Plan(W.Context(many.g.h, many.g.grid_n), many.rec, many.segs)
    W.set_schedule(plan, nbins, 0)
    _print(f"case: {nbins} bins, {plan.info['chunks']} chunks, {dtype}")
    psi, pot, out, ek, ep, ws = _buffers(many, plan, dt)
    W.apply_local_ham(plan, psi, pot, out, ek, ep, workspace=ws)
    torch.cuda.synchronize()
    ref = [t.cpu().numpy().copy() for t in (out, ek, ep)]
    for it in range(20):
        for t in (out, ek, ep):
            t.zero_()
        g = W.Graph(plan, psi, pot, out, ek, ep, workspace=ws)
        g.launch()
        g.close()
        if it % 5 == 4:
            torch.cuda.synchronize()
            for a, t in zip(ref, (out, ek, ep)):
                assert np.array_equal(a, t.cpu().numpy()), it
