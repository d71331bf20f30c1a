"""The LDS limit of the plane kernels when plans of different box sizes are used
at once: it must not follow the last launch.  Two threads, each with its own
context, stream and plan, launch boxes whose back pass needs 107 and 73 KiB
(FP64, 44 and 30 points) or 77 and 64.4 KiB (FP32, 56 and 50 points); every
apply is accepted and gives the bits of the plan used alone.  A graph captured
with the larger boxes replays unchanged after the smaller ones ran."""
import threading

import numpy as np
import pytest

import inputs
from oracle import locreg as LR
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W


def _box_case(n, seed):
    """One box of n^3 points, all of them coarse and a third of them fine."""
    g = inputs.geometry("batch1k", nsf=1)
    g.grid_n = (76, 76, 76)
    rng = np.random.default_rng(seed)
    lo = (8, 8, 8)
    m = np.ones((n, n, n), bool)
    fm = rng.random(m.shape) < 0.3
    om = np.ones((n + 16,) * 3, bool)
    ofm = rng.random(om.shape) < 0.3
    lr = LR.Locreg(lo=lo, dims=(n, n, n), ext=8, cseg=LR.segments_from_mask(m, lo),
                   fseg=LR.segments_from_mask(fm, lo), ocseg=LR.segments_from_mask(om, (0, 0, 0)),
                   ofseg=LR.segments_from_mask(ofm, (0, 0, 0)))
    g.centers = np.zeros((1, 3))
    g.envelope_sigma = np.full(1, 100.0)
    g.domain_lo, g.domain_hi = np.zeros(3), np.array(g.grid_n) * g.h
    return Case(g, [lr])


class _Apply:
    def __init__(self, case, dtype, stream):
        with torch.cuda.stream(stream):
            self.plan = W.Plan(W.Context(case.g.h, case.g.grid_n, stream=stream), case.rec,
                               case.segs)
            self.psi = torch.tensor(case.psi, dtype=dtype, device="cuda")
            self.pot = torch.tensor(case.pot, dtype=dtype, device="cuda")
            self.out = torch.zeros(self.plan.info["out_coefs"], dtype=dtype, device="cuda")
            self.ek = torch.zeros(1, dtype=torch.float64, device="cuda")
            self.ep = torch.zeros_like(self.ek)
            self.ws = self.plan.new_workspace(dtype)
        stream.synchronize()
        self.stream = stream

    def __call__(self):
        W.apply_local_ham(self.plan, self.psi, self.pot, self.out, self.ek, self.ep,
                          workspace=self.ws)

    def result(self):
        self.stream.synchronize()
        return [t.cpu().numpy().copy() for t in (self.out, self.ek, self.ep)]


@pytest.mark.parametrize("dtype,sizes", [("float64", (44, 30)), ("float32", (56, 50))])
def test_threads_with_different_box_sizes(dtype, sizes):
    _print(f"case: two threads, boxes of {sizes} points, {dtype}")
    dt = getattr(torch, dtype)
    runs = [_Apply(_box_case(n, n), dt, torch.cuda.Stream()) for n in sizes]
    alone = []
    for r in runs:
        r()
        alone.append(r.result())
    errors = []

    def work(r, ref):
        try:
            for it in range(150):
                with torch.cuda.stream(r.stream):
                    r()
                if it % 50 == 49:
                    for a, b in zip(ref, r.result()):
                        assert np.array_equal(a, b), it
        except BaseException as e:   # noqa: BLE001 (reported by the main thread)
            errors.append(repr(e))

    ts = [threading.Thread(target=work, args=p) for p in zip(runs, alone)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors


def test_graph_of_large_boxes_after_small_ones():
    _print("case: graph of large boxes, eager small boxes between the replays")
    big, small = (_Apply(_box_case(n, n), torch.float64, torch.cuda.Stream()) for n in (44, 30))
    big()
    ref = big.result()
    g = W.Graph(big.plan, big.psi, big.pot, big.out, big.ek, big.ep, workspace=big.ws)
    for _ in range(3):
        small()
        small.result()
        with torch.cuda.stream(big.stream):
            big.out.zero_()
            g.launch()
        for a, b in zip(ref, big.result()):
            assert np.array_equal(a, b)
    g.close()
