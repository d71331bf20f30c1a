"""The workspace a plan reports: what the kernels of every schedule need and no
more.  The largest schedule is the one with the z part of the kinetic term on
the matrix cores, which takes every function through the nine arrays of the
column kernels, unpadded, plus its energy partials; the plane kernels fit in
that.  A plan that lies just below the static workspace runs in it."""
import numpy as np
import pytest

import inputs
from oracle import locreg as LR
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W


def _up(n, a):
    return (n + a - 1) // a * a


def _arrays(n, e):
    """Elements of the column kernels' arrays of one function."""
    n0, n1, n2 = n
    r0, r1, o0, o1, o2 = 2 * n0 + 29, 2 * n1 + 29, n0 + 2 * e, n1 + 2 * e, n2 + 2 * e
    q = _up(o1, 16)
    return sum(_up(v, 64) for v in (8 * n0 * n1 * n2, 8 * n0 * n1 * n2, 2 * n2 * r0 * r1,
                                    2 * o2 * r0 * r1, 4 * o2 * r0 * q, 8 * n2 * o0 * n1,
                                    8 * n2 * q * n0, 8 * o2 * n0 * n1, 4 * n2 * n1 * r0))


def _partials(n):
    """Energy partials: one per block of k_pot_column, k_kin_col x and y, k_kin_zmfma."""
    n0, n1, n2 = n
    r0, r1 = 2 * n0 + 29, 2 * n1 + 29
    return np.array([-(-r0 * r1 // 256), -(-4 * n1 * n2 // 256), -(-4 * n0 * n2 // 64),
                     -(-n0 * n1 // 16)])


def _case(boxes):
    g = inputs.geometry("batch1k", nsf=1)
    g.grid_n = (90, 90, 50)
    rng = np.random.default_rng(77)
    lrs = []
    for dims, ext in boxes:
        lo = (17, 17, 17)
        m = rng.random((dims[2], dims[1], dims[0])) < 0.9
        m.flat[0] = True
        olo = [max(0, lo[a] - ext) for a in range(3)]
        ohi = [min(g.grid_n[a] - 1, lo[a] + dims[a] - 1 + ext) for a in range(3)]
        om = rng.random((ohi[2] - olo[2] + 1, ohi[1] - olo[1] + 1, ohi[0] - olo[0] + 1)) < 0.9
        lrs.append(LR.Locreg(lo=lo, dims=dims, ext=ext, cseg=LR.segments_from_mask(m, lo),
                             fseg=LR.segments_from_mask(m & (rng.random(m.shape) < 0.3), lo),
                             ocseg=LR.segments_from_mask(om, olo),
                             ofseg=LR.segments_from_mask(om & (rng.random(om.shape) < 0.3), olo)))
    g.centers = np.full((len(lrs), 3), 30 * g.h)
    g.envelope_sigma = np.full(len(lrs), 100.0)
    g.domain_lo, g.domain_hi = np.zeros(3), np.array(g.grid_n) * g.h
    return Case(g, lrs)


# all boxes small; one too wide for the plane kernels in FP64; one in both types
BOXES = {"small": [((20, 21, 22), 8), ((9, 30, 14), 3), ((1, 1, 1), 0)],
         "wide in f64": [((20, 21, 22), 8), ((52, 52, 6), 8)],
         "wide": [((70, 70, 4), 8), ((52, 52, 6), 8), ((11, 12, 13), 8)]}


@pytest.mark.parametrize("name", sorted(BOXES))
def test_reported_workspace(name):
    _print(f"case: reported workspace, {name}")
    boxes = BOXES[name]
    case = _case(boxes)
    plan = W.Plan(W.Context(case.g.h, case.g.grid_n), case.rec, case.segs)
    elems = sum(_arrays(*b) for b in boxes)
    parts = len(boxes) * int(np.max([_partials(d) for d, _ in boxes], axis=0).sum())
    for code, sz in ((W.F32, 4), (W.F64, 8)):
        assert plan.workspace_bytes(code) == _up(elems * sz, 256) + 8 * parts
    # bounded: one function at a time needs the largest function's share
    one = W.Plan(W.Context(case.g.h, case.g.grid_n), case.rec, case.segs, max_workspace=1)
    assert one.info["chunks"] == len(boxes)
    for code, sz in ((W.F32, 4), (W.F64, 8)):
        assert one.workspace_bytes(code) <= _up(max(_arrays(*b) for b in boxes) * sz, 256) + \
            8 * max(int(_partials(d).sum()) for d, _ in boxes)


def test_plan_just_below_the_static_workspace():
    """Eight boxes of 27^3 points without margin: 0.9965 of 128 MiB."""
    _print("case: static apply of a plan just below the static workspace")
    boxes = [((27, 27, 27), 0)] * 8
    case = _case(boxes)
    plan = W.Plan(W.Context(case.g.h, case.g.grid_n), case.rec, case.segs)
    need = _up(8 * _arrays(*boxes[0]) * 8, 256) + 8 * 8 * int(_partials(boxes[0][0]).sum())
    assert plan.workspace_bytes(W.F64) == need and 0.99 * W.STATIC_WORKSPACE_BYTES < need
    psi = torch.tensor(case.psi, dtype=torch.float64, device="cuda")
    pot = torch.tensor(case.pot, dtype=torch.float64, device="cuda")
    outs = []
    for static in (False, True):
        out = torch.zeros(plan.info["out_coefs"], dtype=torch.float64, device="cuda")
        (W.apply_local_ham_static if static else W.apply_local_ham)(plan, psi, pot, out)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
    assert np.any(outs[0]) and np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("name,dtype,points", [("small", "float64", 6), ("wide in f64", "float32", 6),
                                               ("wide in f64", "float64", 12), ("wide", "float32", 12)])
def test_autotuner_tries_the_column_kernels_only_where_a_box_needs_them(name, dtype, points):
    _print(f"case: autotuner candidates, {name}, {dtype}")
    case = _case(BOXES[name])
    dt = getattr(torch, dtype)
    plan = W.Plan(W.Context(case.g.h, case.g.grid_n), case.rec, case.segs)
    psi = torch.tensor(case.psi, dtype=dt, device="cuda")
    pot = torch.tensor(case.pot, dtype=dt, device="cuda")
    out = torch.zeros(plan.info["out_coefs"], dtype=dt, device="cuda")
    best, tried = W.autotune(plan, psi, pot, out, plan.new_workspace(dt), reps=1)
    assert len(tried) == points and best in tried
    assert sorted({t["kin_mfma"] for t in tried}) == ([0] if points == 6 else [0, 1])
