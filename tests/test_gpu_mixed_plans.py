"""Plans whose functions take different kernels: small boxes (plane kernels), one
that fits the LDS in FP32 only (52 x 52 x 6, ext 8: plane kernels in FP32, column
kernels in FP64) and ones past both limits (70 x 70 x 30 and 97 x 9 x 5, more
than 96 points).  Apply (whole, each term, confinement), the accumulating kinetic
call, the synthesis to real space and the schedules with the column kernels,
in one bin, several bins, bounded chunks and a captured step: against the
oracle, and bit for bit against each function alone.  Which kernels ran is
read from the library's launch counts."""
import numpy as np
import pytest

import inputs
from oracle import density as D
from oracle import hamiltonian as Hm
from oracle import locreg as LR
from tests.abi_helpers import rel_err
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W

# dims, ext, types of the plane kernels
BOXES = [((12, 13, 11), 8, "f32 f64"), ((70, 70, 30), 8, ""), ((52, 52, 6), 8, "f32"),
         ((97, 9, 5), 4, ""), ((20, 6, 25), 3, "f32 f64")]


@pytest.fixture(scope="module")
def mixed():
    g = inputs.geometry("batch1k", nsf=1)
    g.grid_n = (118, 90, 50)
    rng = np.random.default_rng(4711)
    lrs = []
    for dims, ext, _ in BOXES:
        lo = tuple(int(rng.integers(ext, g.grid_n[a] - dims[a] - ext + 1)) for a in range(3))
        m = rng.random((dims[2], dims[1], dims[0])) < 0.9
        m.flat[0] = True
        olo = [lo[a] - ext for a in range(3)]
        om = rng.random(tuple(d + 2 * ext for d in dims[::-1])) < 0.9
        lrs.append(LR.Locreg(lo=lo, dims=dims, ext=ext, cseg=LR.segments_from_mask(m, lo),
                             fseg=LR.segments_from_mask(m & (rng.random(m.shape) < 0.3), lo),
                             ocseg=LR.segments_from_mask(om, olo),
                             ofseg=LR.segments_from_mask(om & (rng.random(om.shape) < 0.3), olo),
                             center=tuple((lo[a] + 0.5 * dims[a]) * g.h for a in range(3))))
    g.centers = np.array([l.center for l in lrs])
    g.envelope_sigma = np.full(len(lrs), 100.0)
    g.domain_lo, g.domain_hi = np.zeros(3), np.array(g.grid_n) * g.h
    return Case(g, lrs)


def _alone(case, k):
    one = Case.__new__(Case)
    one.g, one.lrs = case.g, [case.lrs[k]]
    from tests.abi_helpers import to_abi
    one.rec, one.segs = to_abi(one.lrs)
    one.coefs, one.psi, one.pot = [case.coefs[k]], case.coefs[k], case.pot
    return one


def _dt(dtype):
    return torch.float32 if dtype == "f32" else torch.float64


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-5)])
def test_apply(mixed, dtype, tol):
    dt = _dt(dtype)
    n = len(BOXES)
    _print(f"case: mixed plan, {dtype}")
    plan, _, out, ek, ep = mixed.run(dt)
    for k in range(n):
        ref, rk, rp = mixed.oracle(k)
        assert rel_err(out[mixed.out_slice(k)], ref) < tol, k
        assert abs(ek[k] - rk) <= tol * max(1.0, abs(rk)), k
        assert abs(ep[k] - rp) <= tol * max(1.0, abs(rp)), k
        _print(f"  function {k} alone, {BOXES[k][0]}")
        one = _alone(mixed, k)
        ctx = W.Context(one.g.h, one.g.grid_n)
        ctx.profile()
        p1 = W.Plan(ctx, one.rec, one.segs)
        _, _, o1, ek1, ep1 = one.run(dt, plan=p1)
        ran = ctx.profile_read()
        plane = dtype in BOXES[k][2]
        assert ran["back_plane"][0] == int(plane) and ran["back_x"][0] == int(not plane), k
        assert np.array_equal(o1, out[mixed.out_slice(k)]) and ek1[0] == ek[k] and ep1[0] == ep[k]
    # bins, chunks of one function, and chunks of a few
    largest = W.Plan(W.Context(mixed.g.h, mixed.g.grid_n), mixed.rec, mixed.segs,
                     max_workspace=1).workspace_bytes(W.F64)
    for nbins, bound in ((2, 0), (3, 0), (8, 0), (1, 1), (1, largest + (8 << 20))):
        p = W.Plan(W.Context(mixed.g.h, mixed.g.grid_n), mixed.rec, mixed.segs,
                   max_workspace=bound)
        W.set_schedule(p, nbins, 0)
        _, _, o, a, b = mixed.run(dt, plan=p)
        assert np.array_equal(o, out) and np.array_equal(a, ek) and np.array_equal(b, ep), nbins
    # every function on the column kernels
    for nbins in (1, 3):
        W.set_schedule(plan, nbins, 1)
        _, _, o, a, b = mixed.run(dt, plan=plan)
        for k in range(n):
            ref, rk, rp = mixed.oracle(k)
            assert rel_err(o[mixed.out_slice(k)], ref) < tol, k
            assert abs(a[k] - rk) <= tol * max(1.0, abs(rk)), k
            assert abs(b[k] - rp) <= tol * max(1.0, abs(rp)), k


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-5)])
def test_terms_and_graph(mixed, dtype, tol):
    dt = _dt(dtype)
    n = len(BOXES)
    _print(f"case: mixed plan, separate terms and a captured step, {dtype}")
    plan, psi, kin, _, _ = mixed.run(dt, terms=W.KIN)
    _, _, pot, _, _ = mixed.run(dt, terms=W.POT, plan=plan)
    for k in range(n):
        sl = mixed.out_slice(k)
        assert rel_err(kin[sl], mixed.oracle(k, potential=False)[0]) < tol, k
        assert rel_err(pot[sl], mixed.oracle(k, kinetic=False)[0]) < tol, k
    base = torch.ones(plan.info["out_coefs"], dtype=dt, device="cuda")
    W.kinetic(plan, psi, base)
    torch.cuda.synchronize()
    one = np.ones(1, np.float32 if dtype == "f32" else np.float64)
    assert np.array_equal(base.cpu().numpy(), kin + one)
    v = torch.tensor(mixed.pot, dtype=dt, device="cuda")
    bufs = [torch.zeros(plan.info["out_coefs"], dtype=dt, device="cuda")] + \
        [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2)]
    ws = plan.new_workspace(dt)
    W.apply_local_ham(plan, psi, v, *bufs, workspace=ws)
    torch.cuda.synchronize()
    ref = [t.cpu().numpy().copy() for t in bufs]
    g = W.Graph(plan, psi, v, *bufs, workspace=ws)
    for rep in range(3):
        for t in bufs:
            t.zero_()
        g.launch()
        torch.cuda.synchronize()
        for a, t in zip(ref, bufs):
            assert np.array_equal(a, t.cpu().numpy()), rep
    g.close()


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-5)])
def test_confinement_and_synthesis(mixed, dtype, tol):
    dt = _dt(dtype)
    n = len(BOXES)
    _print(f"case: mixed plan, confinement and synthesis, {dtype}")
    plan = W.Plan(W.Context(mixed.g.h, mixed.g.grid_n), mixed.rec, mixed.segs)
    psi = torch.tensor(mixed.psi, dtype=dt, device="cuda")
    v = torch.tensor(mixed.pot, dtype=dt, device="cuda")
    conf = torch.tensor([1e-3, 2e-5, 0.0, 3e-5, 1e-3], dtype=torch.float64, device="cuda")
    out = torch.zeros(plan.info["out_coefs"], dtype=dt, device="cuda")
    ep = torch.zeros(n, dtype=torch.float64, device="cuda")
    W.apply_local_ham(plan, psi, v, out, None, ep, conf=conf)
    fine = torch.zeros(plan.info["fine_box"], dtype=dt, device="cuda")
    W.synthesize(plan, psi, fine)
    torch.cuda.synchronize()
    o, f = out.cpu().numpy(), fine.cpu().numpy()
    off = 0
    for k in range(n):
        ref, _, rp = Hm.apply_local_ham(mixed.lrs[k], mixed.coefs[k], mixed.pot, mixed.g.h,
                                        conf=float(conf[k].item()))
        assert rel_err(o[mixed.out_slice(k)], ref) < tol, k
        assert abs(ep[k].item() - rp) <= tol * max(1.0, abs(rp)), k
        fr = D.fine_values(mixed.lrs[k], mixed.coefs[k]).ravel()
        assert rel_err(f[off:off + fr.size], fr) < tol, k
        off += fr.size
    for nbins, mf in ((3, 0), (1, 1)):
        W.set_schedule(plan, nbins, mf)
        fine.zero_()
        W.synthesize(plan, psi, fine)
        torch.cuda.synchronize()
        f2 = fine.cpu().numpy()
        assert np.array_equal(f2, f) if mf == 0 else rel_err(f2, f) < tol
