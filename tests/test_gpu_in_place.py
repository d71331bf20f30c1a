"""Apply with hpsi written over psi, against the oracle (tolerances of the parity
tests: 1e-12 and 1e-5): patterns that are the same on both sides, functions of
several launch classes, in one chunk and in chunks of one; and, in one chunk, an
output that starts inside the inputs of other functions.  The whole term and each
alone, the accumulating kinetic call, the static workspace and a captured step.
The column kernels have to be the ones that ran, and an apply into a buffer of its
own takes the plane kernels as ever."""
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

BOXES = [(12, 13, 11), (7, 26, 9), (52, 52, 6), (20, 6, 25), (5, 5, 5), (33, 12, 14)]


def _case(ext):
    g = inputs.geometry("batch1k", nsf=1)
    g.grid_n = (90, 90, 50)
    rng = np.random.default_rng(909)
    lrs = []
    for dims in BOXES:
        lo = tuple(int(rng.integers(ext, g.grid_n[a] - dims[a] - ext + 1)) for a in range(3))
        m = rng.random(dims[::-1]) < 0.9
        m.flat[0] = True
        f = m & (rng.random(m.shape) < 0.3)
        c, d = LR.segments_from_mask(m, lo), LR.segments_from_mask(f, lo)
        oc, od = c, d
        if ext:
            olo = [lo[a] - ext for a in range(3)]
            om = rng.random(tuple(n + 2 * ext for n in dims[::-1])) < 0.9
            oc = LR.segments_from_mask(om, olo)
            od = LR.segments_from_mask(om & (rng.random(om.shape) < 0.3), olo)
        lrs.append(LR.Locreg(lo=lo, dims=dims, ext=ext, cseg=c, fseg=d, ocseg=oc, ofseg=od))
    g.centers = np.full((len(lrs), 3), 30 * g.h)
    g.envelope_sigma = np.full(len(lrs), 100.0)
    g.domain_lo, g.domain_hi = np.zeros(3), np.array(g.grid_n) * g.h
    return Case(g, lrs)


@pytest.fixture(scope="module")
def cases():
    return {e: _case(e) for e in (0, 4)}


@pytest.mark.parametrize("ext,bound,shift", [(0, 0, 0), (0, 1, 0), (4, 0, 0), (4, 0, 37)])
@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-5)])
def test_apply_in_place(cases, dtype, tol, ext, bound, shift):
    case, n = cases[ext], len(BOXES)
    dt = torch.float32 if dtype == "f32" else torch.float64
    ctx = W.Context(case.g.h, case.g.grid_n)
    plan = W.Plan(ctx, case.rec, case.segs, max_workspace=bound)
    nin, nout = plan.info["in_coefs"], plan.info["out_coefs"]
    pot = torch.tensor(case.pot, dtype=dt, device="cuda")
    buf = torch.empty(nin + nout, dtype=dt, device="cuda")
    psi, out = buf[shift:shift + nin], buf[:nout]
    assert ext == 0 or nout > nin
    ws = plan.new_workspace(dt)
    ek, ep = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2))

    def fill():
        buf.zero_()
        psi.copy_(torch.tensor(case.psi, dtype=dt))
        ek.zero_(), ep.zero_()

    def check(what, energies=True, **kw):
        torch.cuda.synchronize()
        o = out.cpu().numpy()
        for k in range(n):
            ref, rk, rp = case.oracle(k, **kw)
            assert rel_err(o[case.out_slice(k)], ref) < tol, (what, k)
            if energies:
                assert abs(float(ek[k]) - rk) <= tol * max(1.0, abs(rk)), (what, k)
                assert abs(float(ep[k]) - rp) <= tol * max(1.0, abs(rp)), (what, k)

    _print(f"case: apply in place, {dtype}, ext {ext}, bound {bound}, shift {shift}")
    ctx.profile()
    fill()
    W.apply_local_ham(plan, psi, pot, out, ek, ep, workspace=ws)
    check("whole")
    ran = ctx.profile_read()
    assert ran["back_plane"][0] == 0 and ran["back_x"][0] > 0
    ctx.profile(False)
    for terms, kw in ((W.KIN, dict(potential=False)), (W.POT, dict(kinetic=False))):
        fill()
        W.apply_local_ham(plan, psi, pot, out, workspace=ws, terms=terms)
        check(kw, energies=False, **kw)
    g = W.Graph(plan, psi, pot, out, ek, ep, workspace=ws)
    for rep in range(3):
        fill()
        g.launch()
        check(f"graph {rep}")
    g.close()
    if plan.workspace_bytes(dt) <= W.STATIC_WORKSPACE_BYTES:
        fill()
        W.apply_local_ham_static(plan, psi, pot, out, ek, ep)
        check("static")
    if ext == 0:
        fill()
        W.kinetic(plan, psi, out, workspace=ws)
        torch.cuda.synchronize()
        o = out.cpu().numpy()
        for k in range(n):
            ref = case.oracle(k, potential=False)[0] + case.coefs[k]
            assert rel_err(o[case.out_slice(k)], ref) < tol, k
    ctx.profile()
    ctx.profile_reset()
    fill()
    own = torch.zeros(nout, dtype=dt, device="cuda")
    W.apply_local_ham(plan, psi, pot, own, ek, ep, workspace=ws)
    torch.cuda.synchronize()
    assert ctx.profile_read()["back_plane"][0] > 0
    o = own.cpu().numpy()
    for k in range(n):
        assert rel_err(o[case.out_slice(k)], case.oracle(k)[0]) < tol, k


@pytest.mark.parametrize("ext,bound", [(0, 0), (4, 0)])
@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-5)])
def test_synthesize_in_place(cases, dtype, tol, ext, bound):
    """The values on the fine boxes written over the coefficients, against those in a
    buffer of their own."""
    case = cases[ext]
    dt = torch.float32 if dtype == "f32" else torch.float64
    plan = W.Plan(W.Context(case.g.h, case.g.grid_n), case.rec, case.segs, max_workspace=bound)
    nin, nf = plan.info["in_coefs"], plan.info["fine_box"]
    assert plan.info["chunks"] > 1 and nf > nin
    ws = plan.new_workspace(dt)
    want = torch.zeros(nf, dtype=dt, device="cuda")
    W.synthesize(plan, torch.tensor(case.psi, dtype=dt, device="cuda"), want, workspace=ws)
    _print(f"case: synthesis in place, {dtype}, ext {ext}")
    for at in (0, nf // 2, nf - nin):
        buf = torch.zeros(nf, dtype=dt, device="cuda")
        buf[at:at + nin] = torch.tensor(case.psi, dtype=dt, device="cuda")
        W.synthesize(plan, buf[at:at + nin], buf, workspace=ws)
        torch.cuda.synchronize()
        assert rel_err(buf.cpu().numpy(), want.cpu().numpy()) < tol, at
