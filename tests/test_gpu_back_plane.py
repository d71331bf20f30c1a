"""The forms of the back pass on either side of their lines, alone and mixed in
one plan: in FP32 boxes whose blocks leave room for one per CU take more threads
(57 and 58 points per axis at ext 8, 64 x 64 x 4); boxes of 25 to 32 output rows
take them in one block (not 64 x 16 x 3, which FP64 could no longer take).  Against
the oracle with the bounds of the other parity tests (FP64 1e-12, FP32 1e-5 per
function), and each function of the mixed plan bit for bit as alone, also cut into
bins."""
import numpy as np
import pytest

import inputs
from oracle import locreg as LR
from tests.abi_helpers import rel_err, to_abi
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W

# dims, ext
BOXES = [((57, 57, 3), 8), ((58, 58, 3), 8), ((64, 64, 4), 8), ((96, 30, 2), 8), ((20, 21, 5), 8),
         ((60, 59, 2), 0), ((30, 33, 4), 3),
         ((20, 8, 5), 8), ((20, 9, 5), 8), ((9, 16, 5), 8), ((20, 17, 4), 8), ((96, 10, 3), 8),
         ((64, 16, 3), 8), ((30, 32, 4), 0), ((31, 25, 4), 0), ((17, 26, 5), 3), ((1, 27, 1), 2)]


@pytest.fixture(scope="module")
def case():
    g = inputs.geometry("batch1k", nsf=1)
    g.grid_n = (114, 84, 26)
    rng = np.random.default_rng(99)
    lrs = []
    for dims, ext in BOXES:
        lo = tuple(int(rng.integers(ext, g.grid_n[a] - dims[a] - ext + 1)) for a in range(3))
        m = rng.random(dims[::-1]) < 0.9
        m.flat[0] = True
        om = rng.random(tuple(d + 2 * ext for d in dims[::-1])) < 0.9
        olo = [lo[a] - ext for a in range(3)]
        lrs.append(LR.Locreg(lo=lo, dims=dims, ext=ext, cseg=LR.segments_from_mask(m, lo),
                             fseg=LR.segments_from_mask(m & (rng.random(m.shape) < 0.3), lo),
                             ocseg=LR.segments_from_mask(om, olo),
                             ofseg=LR.segments_from_mask(om & (rng.random(om.shape) < 0.3), olo)))
    g.centers = np.full((len(lrs), 3), 20 * g.h)
    g.envelope_sigma = np.full(len(lrs), 100.0)
    g.domain_lo, g.domain_hi = np.zeros(3), np.array(g.grid_n) * g.h
    return Case(g, lrs)


@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 1e-5)])
def test_back_pass_forms(case, dtype, tol):
    dt = getattr(torch, dtype)
    _print(f"case: forms of the back pass, {dtype}")
    plan, _, out, ek, ep = case.run(dt)
    _, _, kin, _, _ = case.run(dt, terms=W.KIN, plan=plan)
    for k in range(len(BOXES)):
        ref, rk, rp = case.oracle(k)
        sl = case.out_slice(k)
        assert rel_err(out[sl], ref) < tol, k
        assert rel_err(kin[sl], case.oracle(k, potential=False)[0]) < tol, k
        assert abs(ek[k] - rk) <= tol * max(1.0, abs(rk)), k
        assert abs(ep[k] - rp) <= tol * max(1.0, abs(rp)), k
        _print(f"  box {BOXES[k]} alone")
        one = Case.__new__(Case)
        one.g, one.lrs = case.g, [case.lrs[k]]
        one.rec, one.segs = to_abi(one.lrs)
        one.coefs, one.psi, one.pot = [case.coefs[k]], case.coefs[k], case.pot
        _, _, o1, ek1, ep1 = one.run(dt)
        assert np.array_equal(o1, out[sl]) and ek1[0] == ek[k] and ep1[0] == ep[k], k
    for nbins in (2, 4):
        W.set_schedule(plan, nbins, 0)
        _, _, o, a, b = case.run(dt, plan=plan)
        assert np.array_equal(o, out) and np.array_equal(a, ek) and np.array_equal(b, ep), nbins
