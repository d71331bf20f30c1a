"""S and H values with eight, four and two waves per pair: the largest and the
smallest patterns of each, on boxes whose rows hold several runs and whose pairs
have more rows than one batch of 64.  Against the product of the functions' dense
coefficient vectors in FP64; the products of FP32 inputs are exact in double, so
both types keep 1e-12 of the norms (sums of fewer than 2^13 terms: 2^13 2^-53)."""
import numpy as np
import pytest

import inputs
from oracle import locreg as LR
from tests.test_gpu_parity import Case, _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _case(nsf, dims, ext):
    g = inputs.geometry("batch1k", nsf=nsf)
    g.grid_n = (40, 40, 40)
    rng = np.random.default_rng(nsf)
    lrs = []
    for k in range(nsf):
        lo = tuple(int(v) for v in rng.integers(6, 8, 3))
        m = rng.random((dims[2], dims[1], dims[0])) >= 0.2
        m.flat[0] = True
        m[1:, 1:, 1:].flat[0] = True   # a point that every function has
        m[-2:, -2:, -2:] = True
        olo = [lo[a] - ext for a in range(3)]
        om = rng.random(tuple(dims[a] + 2 * ext for a in (2, 1, 0))) >= 0.2
        om[ext:-ext, ext:-ext, ext:-ext] |= m
        lrs.append(LR.Locreg(lo=lo, dims=dims, ext=ext, cseg=LR.segments_from_mask(m, lo),
                             fseg=LR.segments_from_mask(m & (rng.random(m.shape) < 0.5), lo),
                             ocseg=LR.segments_from_mask(om, olo),
                             ofseg=LR.segments_from_mask(om & (rng.random(om.shape) < 0.5), olo)))
    g.centers, g.envelope_sigma = np.zeros((nsf, 3)), np.full(nsf, 100.0)
    g.domain_lo, g.domain_hi = np.zeros(3), np.array(g.grid_n) * g.h
    return Case(g, lrs)


def _dense(case, v, out):
    """Coefficient vectors v (the layout of one pattern) on the whole grid."""
    n = case.g.grid_n[0]
    pre = "o" if out else ""
    D = np.zeros((len(case.lrs), 8, n, n, n))
    for k, r in enumerate(case.rec):
        o, nc = int(r[pre + "coef_off"]), int(r["on_c" if out else "n_c"])
        for c, kind in enumerate("cf"):
            a = int(r[pre + "seg_" + kind])
            for s in case.segs[a:a + int(r["n" + pre + "seg_" + kind])]:
                x0, x1, y, z, off = (int(s[f]) for f in ("i1s", "i1e", "i2", "i3", "off"))
                m = x1 - x0 + 1
                if c == 0:
                    D[k, 0, z, y, x0:x1 + 1] = v[o + off:o + off + m]
                else:
                    q = v[o + nc + 7 * off:o + nc + 7 * (off + m)].reshape(m, 7)
                    D[k, 1:, z, y, x0:x1 + 1] = q.T
    return D.reshape(len(case.lrs), -1)


@pytest.mark.parametrize("nsf", [3, 64, 65, 181, 182])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_sparse_values_by_waves(nsf, dtype):
    """Every pair shares points: nsf^2 entries (4,096 / 4,225 and 32,761 /
    33,124 lie on either side of the two lines)."""
    _print(f"case: sparse values, {nsf} boxes, {dtype}")
    import paper_1401_7441_amd as W
    case = _case(nsf, (7, 9, 10) if nsf < 100 else (6, 4, 3), 1)
    plan = W.Plan(W.Context(case.g.h, case.g.grid_n), case.rec, case.segs)
    rng = np.random.default_rng(3)
    data = [torch.tensor(rng.standard_normal(plan.info[c]), dtype=dtype)
            for c in ("in_coefs", "out_coefs")]
    dev = [t.cuda() for t in data]
    bra = _dense(case, data[0].double().numpy(), False)
    for out in (False, True):
        ket = _dense(case, data[1].double().numpy(), True) if out else bra
        want = bra @ ket.T
        scale = np.linalg.norm(bra, axis=1)[:, None] * np.linalg.norm(ket, axis=1)[None, :]
        rp, cl, val = W.sparse_overlap(plan, dev[0], dev[1] if out else dev[0], out)
        rp, cl, v = rp.cpu().numpy(), cl.cpu().numpy(), val.cpu().numpy()
        assert len(v) == nsf * nsf
        rows = np.repeat(np.arange(nsf), np.diff(rp))
        assert np.max(np.abs(v - want[rows, cl]) / scale[rows, cl]) <= 1e-12
        if not out:   # each pair once and mirrored, or every pair: the same bits
            _, _, w = W.sparse_overlap(plan, dev[0], dev[0].clone(), False)
            assert np.array_equal(w.cpu().numpy(), v)
            assert np.array_equal(v.reshape(nsf, nsf), v.reshape(nsf, nsf).T)
