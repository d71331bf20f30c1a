"""wvl_density with infinite and NaN values: they enter the entries of K that
name their function and no others.  40 and 150 functions (one and several chunks
per tile) with positive values and a sparse positive K; against the entries
summed one by one in numpy (a box that does not meet a tile's plane of 16 x 4 x 1
points takes no part there).  The finite densities agree to the bounds of the
other density tests, and are those without the planted values."""
import numpy as np
import pytest

from oracle import locreg as LR
from tests.abi_helpers import to_abi
from tests.test_gpu_density import TOL
from tests.test_gpu_parity import _print

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W

GRID = (18, 18, 18)
GF = tuple(2 * n + 29 for n in GRID)


def _system(nsf, seed):
    rng = np.random.default_rng(seed)
    lrs = []
    for k in range(nsf):
        lo = tuple(int(v) for v in rng.integers(0, 15, 3))
        dims = tuple(int(v) for v in rng.integers(1, 4, 3))
        if k % 10 in (4, 5, 6):            # these three share a box and entries
            lo, dims = (5, 6, 7), (2, 2, 2)
        lrs.append(LR.box_locreg(lo, dims, lo, lo))
    fine = [rng.uniform(0.5, 1.5, [2 * d + 29 for d in l.dims[::-1]]) for l in lrs]
    K = {}
    for a in range(nsf):
        group = a % 10 in (4, 5, 6)
        K[a, a] = rng.uniform(0.5, 1.0)
        for b in rng.integers(0, nsf, 6):
            if group == (b % 10 in (4, 5, 6)) and (not group or a // 10 == b // 10):
                K[a, int(b)] = rng.uniform(0.5, 1.0)
    return lrs, fine, K


def _reference(lrs, fine, K):
    """Sum over the entries, on the tile planes that both boxes meet."""
    rho = np.zeros(GF[::-1])
    tile = (16, 4, 1)
    for (a, b), k in K.items():
        A, B = lrs[a], lrs[b]
        sl = []
        for d in range(3):
            lo, hi = 0, GF[d]
            for L in (A, B):
                o, r = 2 * L.lo[d], 2 * L.dims[d] + 29
                lo, hi = max(lo, o // tile[d] * tile[d]), min(hi, -(-(o + r) // tile[d]) * tile[d])
            sl.append((lo, hi))
        if any(lo >= hi for lo, hi in sl):
            continue
        vals = []
        for L, f in ((A, fine[a]), (B, fine[b])):
            v = np.zeros([hi - lo for lo, hi in sl][::-1])
            src, dst = [], []
            for d in (2, 1, 0):
                o, r = 2 * L.lo[d], 2 * L.dims[d] + 29
                x0, x1 = max(sl[d][0], o), min(sl[d][1], o + r)
                src.append(slice(x0 - o, x1 - o))
                dst.append(slice(x0 - sl[d][0], x1 - sl[d][0]))
            v[tuple(dst)] = f[tuple(src)]
            vals.append(v)
        with np.errstate(invalid="ignore"):
            rho[tuple(slice(*sl[d]) for d in (2, 1, 0))] += vals[0] * (k * vals[1])
    return rho


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nsf", [40, 150])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_values_enter_their_entries_only(nsf, dtype, value):
    _print(f"case: density, {nsf} functions, {value}, {dtype}")
    lrs, fine, K = _system(nsf, nsf)
    dt = torch.float64 if dtype == "f64" else torch.float32
    if dtype == "f32":
        fine = [f.astype(np.float32).astype(np.float64) for f in fine]
    clean = _reference(lrs, fine, K)
    # an explicit zero entry, in the row of a function with a smaller index
    q = nsf - 15            # nsf = 40, 150: index 5 of its group of ten
    assert q % 10 == 5
    K[q - 1, q] = 0.0
    clean0 = _reference(lrs, fine, K)
    fine[q][3, 4, 5] = value
    fine[5][10, 11, 12] = value
    want = _reference(lrs, fine, K)
    plan = W.Plan(W.Context(0.45, GRID), *to_abi(lrs))
    ent = sorted(K)
    rp = np.searchsorted([a for a, _ in ent], np.arange(nsf + 1))
    args = (torch.tensor(rp, dtype=torch.int64, device="cuda"),
            torch.tensor([b for _, b in ent], dtype=torch.int32, device="cuda"),
            torch.tensor([K[e] for e in ent], dtype=torch.float64, device="cuda"))
    f = torch.tensor(np.concatenate([x.ravel() for x in fine]), dtype=dt, device="cuda")
    rho = torch.zeros(int(np.prod(GF)), dtype=dt, device="cuda")
    W.density(plan, f, *args, rho)
    torch.cuda.synchronize()
    got = rho.cpu().numpy().astype(np.float64).reshape(want.shape)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isinf(got), np.isinf(want))
    fin = np.isfinite(want)
    assert (~fin).sum() == 2
    assert np.max(np.abs(got[fin] - want[fin])) <= TOL[dtype] * np.max(np.abs(clean))
    assert np.array_equal(want[fin], clean0[fin])
    # the second planted value has no zero entry: infinite, not NaN
    p = [2 * lrs[5].lo[d] + (12, 11, 10)[d] for d in range(3)]
    assert np.isinf(want[p[2], p[1], p[0]]) == np.isinf(value)
