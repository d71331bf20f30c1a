"""Infinite and NaN values in the coefficients and in the potential: they reach
the outputs whose taps meet them and no others, also where the passes are
products with banded matrices.  The column kernels (the schedule with kin_mfma),
which form every output from its taps alone, are the reference: the same outputs
are finite, with the same values (FP32: the same bits; FP64 1e-12), and the
energies are of the same kind."""
import numpy as np
import pytest

from tests.test_gpu_parity import _print
from tests.test_gpu_planes import _case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W


def _same(a, b, exact):
    """The same values are finite, and these agree."""
    fa, fb = np.isfinite(a), np.isfinite(b)
    assert np.array_equal(fa, fb), (int((~fa).sum()), int((~fb).sum()))
    if exact:
        assert np.array_equal(a[fa], b[fb])
    else:
        assert np.linalg.norm(a[fa] - b[fb]) <= 1e-12 * np.linalg.norm(b[fb])
    return int((~fa).sum())


def _kind(x):
    return "nan" if np.isnan(x) else "inf" if np.isinf(x) else "finite"


def _run(plan, psi, pot, dt, terms):
    out = torch.zeros(plan.info["out_coefs"], dtype=dt, device="cuda")
    ek = torch.zeros(1, dtype=torch.float64, device="cuda")
    ep = torch.zeros_like(ek)
    W.apply_local_ham(plan, psi, pot, out, ek, ep, terms=terms)
    fine = torch.zeros(plan.info["fine_box"], dtype=dt, device="cuda")
    W.synthesize(plan, psi, fine)
    torch.cuda.synchronize()
    return out.cpu().numpy(), ek.item(), ep.item(), fine.cpu().numpy()


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("where", ["coarse", "wavelet", "last", "potential", "potential edge"])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_non_finite_values_keep_to_their_taps(dtype, where, value):
    _print(f"case: {value} in {where}, {dtype}")
    dt = getattr(torch, dtype)
    dims, ext = (41, 44, 47), 8
    case = _case(dims, ext)
    psi = torch.tensor(case.psi, dtype=dt, device="cuda")
    pot = torch.tensor(case.pot, dtype=dt, device="cuda")
    r = case.rec[0]
    if where == "coarse":
        psi[int(r["n_c"]) // 2] = value
    elif where == "wavelet":
        psi[int(r["n_c"]) + 7 * (int(r["n_f"]) // 2) + 3] = value
    elif where == "last":
        psi[-1] = value
    else:
        p = [2 * int(r["lo"][a]) + (dims[a] + 14 if where == "potential" else 0) for a in range(3)]
        pot.view(case.pot.shape)[p[2], p[1], p[0]] = value
    plan = W.Plan(W.Context(case.g.h, case.g.grid_n), case.rec, case.segs)
    out, _, ep, fine = _run(plan, psi, pot, dt, W.POT)
    kin, ek, _, _ = _run(plan, psi, pot, dt, W.KIN)
    full, _, _, _ = _run(plan, psi, pot, dt, W.KIN | W.POT)
    W.set_schedule(plan, 1, 1)
    ref, _, rp, rfine = _run(plan, psi, pot, dt, W.POT)
    bad = _same(out, ref, dtype == "float32")
    badf = _same(fine, rfine, dtype == "float32")
    _print(f"  {bad} of {out.size} outputs, {badf} of {fine.size} fine values not finite")
    assert 0 < bad < out.size and (badf > 0) == (not where.startswith("potential"))
    assert _kind(ep) == _kind(rp) != "finite"
    # the kinetic term: 29 taps per axis, none of them elsewhere
    assert np.array_equal(np.isfinite(full), np.isfinite(ref) & np.isfinite(kin))
    assert np.isfinite(ek) == where.startswith("potential")
    assert np.all(np.isfinite(kin)) == where.startswith("potential")
