"""wvl_density at the edges of its function chunks (64) and point tiles, with a
kernel that is neither symmetric nor free of duplicated entries: against the
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
@pytest.mark.parametrize("nsf", [1, 16, 63, 64, 65, 129])
def test_density_chunk_edges(nsf, dtype):
    _print(f"case: density, {nsf} functions, {dtype}")
    rng = np.random.default_rng(nsf)
    lrs = []
    for _ in range(nsf):
        lo = tuple(int(v) for v in rng.integers(7, 10, 3))
        dims = tuple(int(v) for v in rng.integers(1, 4, 3))
        lrs.append(LR.box_locreg(lo, dims, lo, lo))
    g1 = inputs.geometry("single")
    case = Case(dataclasses.replace(g1, centers=np.repeat(g1.centers, nsf, axis=0),
                                    radii=np.repeat(g1.radii, nsf),
                                    fine_radii=np.repeat(g1.fine_radii, nsf),
                                    envelope_sigma=np.repeat(g1.envelope_sigma, nsf)), lrs)
    # rows of up to 300 entries: every column, many of them twice or more
    rp, cl, val, K = [0], [], [], np.zeros((nsf, nsf))
    for a in range(nsf):
        cols = rng.integers(0, nsf, int(rng.integers(0, 300)))
        v = rng.standard_normal(len(cols))
        np.add.at(K[a], cols, v)
        cl.append(cols)
        val.append(v)
        rp.append(rp[-1] + len(cols))
    dt = torch.float64 if dtype == "f64" else torch.float32
    plan, psi, fine = _synth(case, dt)
    n = case.g.grid_n
    size = (2 * n[2] + 29) * (2 * n[1] + 29) * (2 * n[0] + 29)
    args = (torch.tensor(rp, dtype=torch.int64, device="cuda"),
            torch.tensor(np.concatenate(cl), dtype=torch.int32, device="cuda"),
            torch.tensor(np.concatenate(val), device="cuda"))
    got = []
    for _ in range(3):
        rho = torch.full((size,), float("nan"), dtype=dt, device="cuda")
        W.density(plan, fine, *args, rho)
        torch.cuda.synchronize()
        got.append(rho.cpu().numpy())
    want = D.density(case.lrs, case.coefs, K, n).ravel()
    assert np.max(np.abs(got[0] - want)) <= TOL[dtype] * max(np.max(np.abs(want)), 1e-300)
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
