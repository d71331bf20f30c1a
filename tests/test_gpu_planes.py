"""The plane kernels of the local Hamiltonian at the edges of their tiles: box
edges around 16-point tiles, 24-row strips, 32-lane rows and the LDS limit,
every kind of output margin, random patterns of many runs per row.

Against the oracle with the bounds of the other parity tests (FP64 1e-12,
FP32 1e-5 relative per function).  In FP32 the potential part has the operation
order of the column kernels (the schedule with the z kinetic part on the
matrix cores runs those), so it and its energy are compared bit for bit."""
import numpy as np
import pytest

import inputs
from oracle import locreg as LR
from tests.abi_helpers import rel_err
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W

# dims (x, y, z), ext
BOXES = [((1, 1, 1), 0), ((2, 17, 3), 3), ((8, 9, 16), 8), ((32, 8, 9), 1), ((33, 32, 2), 8),
         ((34, 33, 4), 16), ((25, 40, 3), 7), ((50, 49, 2), 8), ((67, 12, 3), 5), ((5, 7, 52), 8)]


def _case(dims, ext):
    g = inputs.geometry("batch1k", nsf=1)
    g.grid_n = (84, 84, 84)
    rng = np.random.default_rng(sum(dims) + 100 * ext)
    lo = (9, 12, 14)
    m = rng.random((dims[2], dims[1], dims[0])) < 0.85
    m.flat[0] = True
    olo = [max(0, lo[a] - ext) for a in range(3)]
    ohi = [min(g.grid_n[a] - 1, lo[a] + dims[a] - 1 + ext) for a in range(3)]
    om = rng.random((ohi[2] - olo[2] + 1, ohi[1] - olo[1] + 1, ohi[0] - olo[0] + 1)) < 0.9
    lr = LR.Locreg(lo=lo, dims=dims, ext=ext, cseg=LR.segments_from_mask(m, lo),
                   fseg=LR.segments_from_mask(m & (rng.random(m.shape) < 0.5), lo),
                   ocseg=LR.segments_from_mask(om, olo),
                   ofseg=LR.segments_from_mask(om & (rng.random(om.shape) < 0.6), olo))
    g.centers = np.array([[h * g.h for h in lo]], dtype=float)
    g.envelope_sigma = np.full(1, 100.0)
    g.domain_lo, g.domain_hi = np.zeros(3), np.array(g.grid_n) * g.h
    return Case(g, [lr])


@pytest.mark.parametrize("dims,ext", BOXES)
def test_plane_kernels(dims, ext):
    _print(f"case: box {dims}, ext {ext}")
    case = _case(dims, ext)
    ref, rk, rp = case.oracle(0)
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 1e-5)):
        _, _, out, ek, ep = case.run(dtype)
        assert rel_err(out[case.out_slice(0)], ref) < tol
        assert abs(ek[0] - rk) <= tol * max(1.0, abs(rk)) and abs(ep[0] - rp) <= tol * max(1.0, abs(rp))
    _, _, kin, _, _ = case.run(torch.float64, terms=W.KIN)
    assert rel_err(kin[case.out_slice(0)], case.oracle(0, potential=False)[0]) < 1e-12
    # FP32, potential part: the bits of the column kernels
    plan, _, a, _, ea = case.run(torch.float32, terms=W.POT)
    W.set_schedule(plan, 1, 1)
    _, _, b, _, eb = case.run(torch.float32, terms=W.POT, plan=plan)
    assert np.array_equal(a, b) and np.array_equal(ea, eb)


@pytest.mark.parametrize("n", [8, 9])
def test_up_and_kinetic_in_one_launch(n):
    """Eight of these boxes have 944 blocks of the up pass and the z part (one
    launch, at most 1,024), nine have 1,062 (two launches)."""
    one = _case((5, 7, 52), 8)
    g = one.g
    g.centers = np.repeat(g.centers, n, axis=0)
    g.envelope_sigma = np.full(n, 100.0)
    case = Case(g, [one.lrs[0]] * n)
    _print(f"case: {n} boxes (5, 7, 52)")
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 1e-5)):
        _, _, out, ek, ep = case.run(dtype)
        for k in (0, n - 1):
            ref, rk, rp = case.oracle(k)
            assert rel_err(out[case.out_slice(k)], ref) < tol
            assert abs(ek[k] - rk) <= tol * max(1.0, abs(rk))
            assert abs(ep[k] - rp) <= tol * max(1.0, abs(rp))
