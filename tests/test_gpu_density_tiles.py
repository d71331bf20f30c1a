"""wvl_density on either side of the line between tiles of few and of many
functions (32), with kernels that leave whole 16 x 16 blocks of a tile's functions
without an entry (diagonal; groups of 16 and of 5; one row only): against the
oracle (FP64 1e-12, FP32 1e-5 of the largest value, the bounds of the other
density tests), and bit for bit the same when run again."""
import dataclasses

import numpy as np
import pytest

import inputs
from oracle import density as D
from oracle import locreg as LR
from tests.test_gpu_density import TOL, _synth
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nsf", [31, 32, 33, 80])
def test_density_by_cover_and_blocks(nsf, dtype):
    rng = np.random.default_rng(nsf)
    lrs = []
    for _ in range(nsf):
        lo = tuple(int(v) for v in rng.integers(7, 10, 3))
        lrs.append(LR.box_locreg(lo, tuple(int(v) for v in rng.integers(1, 4, 3)), lo, lo))
    # one far off: tiles that a single function or none meets
    lrs[-1] = LR.box_locreg((30, 30, 30), (2, 2, 2), (30, 30, 30), (30, 30, 30))
    g1 = inputs.geometry("single")
    g1.grid_n = (40, 40, 40)
    case = Case(dataclasses.replace(g1, centers=np.repeat(g1.centers, nsf, axis=0),
                                    radii=np.repeat(g1.radii, nsf),
                                    fine_radii=np.repeat(g1.fine_radii, nsf),
                                    envelope_sigma=np.repeat(g1.envelope_sigma, nsf)), lrs)
    dt = torch.float64 if dtype == "f64" else torch.float32
    plan, psi, fine = _synth(case, dt)
    n = case.g.grid_n
    idx = np.arange(nsf)
    for kind, mask in (("diagonal", idx[:, None] == idx), ("groups of 16", idx[:, None] // 16 == idx // 16),
                       ("groups of 5", idx[:, None] // 5 == idx // 5), ("one row", (idx == 7)[:, None] & (idx >= 0)),
                       ("last column", (idx == nsf - 2) & (idx >= 0)[:, None])):
        _print(f"case: density, {nsf} functions, {kind}, {dtype}")
        K = rng.standard_normal((nsf, nsf)) * mask
        rows, cols = np.nonzero(mask)
        args = (torch.tensor(np.searchsorted(rows, np.arange(nsf + 1)), device="cuda"),
                torch.tensor(cols.astype(np.int32), device="cuda"),
                torch.tensor(K[rows, cols], device="cuda"))
        got = []
        for _ in range(2):
            rho = torch.full(((2 * n[2] + 29) * (2 * n[1] + 29) * (2 * n[0] + 29),), float("nan"),
                             dtype=dt, device="cuda")
            W.density(plan, fine, *args, rho)
            torch.cuda.synchronize()
            got.append(rho.cpu().numpy())
        want = D.density(case.lrs, case.coefs, K, n).ravel()
        assert np.max(np.abs(got[0] - want)) <= TOL[dtype] * max(np.max(np.abs(want)), 1e-300), kind
        assert np.array_equal(got[0], got[1]), kind
