"""S and H values do not depend on the plan they are formed in: the pairs of
six functions have the same bits when the plan holds them alone (at most 36
entries), with 65 and with 182 coinciding small functions elsewhere (4,225 and
33,124 more entries),
and with one pair only; the number of waves per pair differs in these.  Boxes of
4 to 30 points per axis: pairs of one to more than eight batches of 64 rows."""
import numpy as np
import pytest

from oracle import locreg as LR
from tests.abi_helpers import to_abi
from tests.test_gpu_parity import _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W


def _functions():
    rng = np.random.default_rng(31)
    lrs = []
    for n in (30, 28, 12, 25, 4, 9):
        lo = tuple(int(v) for v in rng.integers(10, 16, 3))
        m = rng.random((n, n, n)) < 0.9
        m.flat[0] = True
        om = rng.random((n + 4,) * 3) < 0.9
        olo = tuple(v - 2 for v in lo)
        lrs.append(LR.Locreg(lo=lo, dims=(n, n, n), ext=2, cseg=LR.segments_from_mask(m, lo),
                             fseg=LR.segments_from_mask(m & (rng.random(m.shape) < 0.4), lo),
                             ocseg=LR.segments_from_mask(om, olo),
                             ofseg=LR.segments_from_mask(om & (rng.random(om.shape) < 0.4), olo)))
    return lrs


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_pair_values_are_those_of_every_plan(dtype):
    dt = getattr(torch, dtype)
    fns = _functions()
    small = LR.box_locreg((55, 55, 55), (2, 2, 2), (55, 55, 55), (55, 55, 55))
    rng = np.random.default_rng(5)
    psi = [rng.standard_normal(l.n_c + 7 * l.n_f) for l in fns]
    hpsi = [rng.standard_normal(l.on_c + 7 * l.on_f) for l in fns]

    def values(keep, extra):
        _print(f"case: S and H of functions {keep} with {extra} others, {dtype}")
        lrs = [fns[k] for k in keep] + [small] * extra
        p = np.concatenate([psi[k] for k in keep] + [np.ones(15)] * extra)
        h = np.concatenate([hpsi[k] for k in keep] + [np.ones(15)] * extra)
        plan = W.Plan(W.Context(0.45, (60, 60, 60)), *to_abi(lrs))
        p, h = (torch.tensor(v, dtype=dt, device="cuda") for v in (p, h))
        out = []
        for ket, ket_out in ((p, False), (p.clone(), False), (h, True)):
            rp, cl, val = (t.cpu().numpy() for t in W.sparse_overlap(plan, p, ket, ket_out))
            n = len(keep)
            full = np.zeros((n, n))   # pairs that share no point: 0
            for a in range(n):
                full[a, cl[rp[a]:rp[a + 1]]] = val[rp[a]:rp[a + 1]]
            assert len(cl) == np.count_nonzero(full) + extra ** 2
            out.append(full)
        return out

    ref = values(range(6), 0)
    assert np.array_equal(ref[0], ref[1]) and np.array_equal(ref[0], ref[0].T)
    for extra in (65, 182):
        for a, b in zip(ref, values(range(6), extra)):
            assert np.array_equal(a, b), extra
    for pair in ((0, 1), (2, 5)):
        for a, b in zip(ref, values(pair, 0)):
            assert np.array_equal(a[np.ix_(pair, pair)], b), pair


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("rows,counts", [(17, (59, 60, 84, 100, 255, 256, 363)), (15, (60, 256)),
                                         (10, (60, 182, 256)), (6, (100,))])
def test_every_number_of_waves(rows, counts, dtype):
    """n boxes of 3 x rows x rows points in one place, n^2 H entries and n (n + 1) / 2
    sums of S, around each line of the rule for the waves per pair: the Gram
    matrices of the coefficients (FP64 1e-12 of the norms; products of FP32 values
    are exact in double), and the three first functions' bits as in a plan of
    their own."""
    dt = getattr(torch, dtype)
    box = LR.box_locreg((4, 4, 4), (3, rows, rows), (4, 5, 5), (6, rows + 1, rows + 1))
    m = box.n_c + 7 * box.n_f
    rng = np.random.default_rng(rows)
    data = torch.tensor(rng.standard_normal((2, max(counts), m)), dtype=dt)
    small = None
    for n in (3,) + counts:
        _print(f"case: {n} boxes of {rows * rows} rows, {dtype}")
        plan = W.Plan(W.Context(0.45, (40, 40, 40)), *to_abi([box] * n))
        p, h = (data[k, :n].contiguous().cuda() for k in (0, 1))
        got = []
        for ket, ket_out in ((p, False), (h, True)):
            _, cl, val = W.sparse_overlap(plan, p.view(-1), ket.view(-1), ket_out)
            assert len(cl) == n * n
            v = val.cpu().numpy().reshape(n, n)
            a, b = (t.double().cpu().numpy() for t in (p, ket))
            scale = np.linalg.norm(a, axis=1)[:, None] * np.linalg.norm(b, axis=1)[None, :]
            assert np.max(np.abs(v - a @ b.T) / scale) <= 1e-12
            got.append(v[:3, :3].copy())
        small = small or got
        for a, b in zip(small, got):
            assert np.array_equal(a, b), n
