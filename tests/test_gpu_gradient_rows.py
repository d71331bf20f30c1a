"""wvl_gradient where its row lists can go wrong: rows of several runs on
every pattern (lists longer than one round), more neighbours than lanes, and
rows of more than 256 wavelet values.  Against the oracle, FP64 1e-12 and FP32
1e-5 relative per function (the bounds of the other gradient tests)."""
import numpy as np
import pytest

import inputs
from oracle import gradient as G
from oracle import locreg as LR
from tests.abi_helpers import rel_err
from tests.test_gpu_gradient import _dense, _run
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _case(nsf, dims, ext, hole):
    """nsf boxes a point or two apart, every pattern random with a share `hole`
    of its points left out (corner and diagonal kept)."""
    g = inputs.geometry("batch1k", nsf=nsf)
    g.grid_n = (64, 40, 40)
    rng = np.random.default_rng(nsf + 10 * ext)
    lrs = []
    for k in range(nsf):
        lo = tuple(int(v) for v in rng.integers(6, 9, 3))
        m = rng.random((dims[2], dims[1], dims[0])) >= hole
        m.flat[0] = True
        olo = [lo[a] - ext for a in range(3)]
        om = rng.random(tuple(dims[a] + 2 * ext for a in (2, 1, 0))) >= hole
        om[ext:-ext or None, ext:-ext or None, ext:-ext or None] |= m
        lrs.append(LR.Locreg(lo=lo, dims=dims, ext=ext, cseg=LR.segments_from_mask(m, lo),
                             fseg=LR.segments_from_mask(m & (rng.random(m.shape) >= hole), lo),
                             ocseg=LR.segments_from_mask(om, olo),
                             ofseg=LR.segments_from_mask(om & (rng.random(om.shape) >= hole), olo)))
    g.centers, g.envelope_sigma = np.zeros((nsf, 3)), np.full(nsf, 100.0)
    g.domain_lo, g.domain_hi = np.zeros(3), np.array(g.grid_n) * g.h
    return Case(g, lrs)


@pytest.mark.parametrize("nsf,dims,ext,hole", [(70, (7, 3, 2), 2, 0.3), (5, (41, 2, 2), 1, 0.0),
                                               (9, (40, 3, 1), 0, 0.4)])
def test_gradient_rows(nsf, dims, ext, hole):
    _print(f"case: gradient rows, {nsf} boxes {dims}, ext {ext}")
    case = _case(nsf, dims, ext, hole)
    import paper_1401_7441_amd as W
    ctx = W.Context(case.g.h, case.g.grid_n)
    plan = W.Plan(ctx, case.rec, case.segs)
    pats = []
    for out in (False, True):
        n = W.sparse_pattern_nnz(plan, out)
        z = torch.zeros(max(plan.info["in_coefs"], plan.info["out_coefs"]), dtype=torch.float64,
                        device="cuda")
        rp, cl, _ = W.sparse_overlap(plan, z, z, out, values=False)
        pats.append((rp.cpu().numpy(), cl.cpu().numpy()))
        assert n == len(pats[-1][1])
    rng = np.random.default_rng(7)
    (srp, scl), (hrp, hcl) = pats
    mask = _dense(nsf, srp, scl, np.ones(len(scl))) > 0
    S0, H0, K0 = (rng.standard_normal((nsf, nsf)) * 0.1 for _ in range(3))
    S0, H0, K0 = (0.5 * (x + x.T) for x in (S0 + np.eye(nsf), H0, K0))
    vals = lambda A, rp, cl: np.array([A[a, cl[q]] for a in range(nsf)  # noqa: E731
                                       for q in range(rp[a], rp[a + 1])])
    hpsi = [rng.standard_normal(l.on_c + 7 * l.on_f) for l in case.lrs]
    A, M = G.coefficient_matrices(S0 * mask, H0, K0 * mask, mask)
    want = G.gradient(case.lrs, case.coefs, hpsi, A, M, mask)
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 1e-5)):
        _, got = _run(case, case.coefs, hpsi, vals(S0, srp, scl), vals(H0, hrp, hcl),
                      vals(K0, srp, scl), dtype)
        for k, l in enumerate(case.lrs):
            o = int(case.rec[k]["coef_off"])
            assert rel_err(got[o:o + len(want[k])], want[k]) < tol, k
