"""Products of the Fermi operator expansion from rows spread out in LDS, on both
sides of the line where a block takes one row (160 KiB of LDS hold four blocks)
or several: 317 and 318 equal groups of 16 functions whose rows differ in length,
and 400 with two blocks left per CU and rows that are not a multiple of the blocks.
Groups share no points, so K and mu of each are those of one group with its share
of the occupation, with the same bits in every group.  Oracle and tolerances as in
test_gpu_foe."""
import numpy as np
import pytest

from oracle import foe as F
from oracle import locreg as LR
from tests.abi_helpers import to_abi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1401_7441_amd as W
    from tests.test_gpu_foe import _tolerances


@pytest.mark.parametrize("groups", [317, 318, 400])
def test_rows_per_block(groups):
    m, sizes = 16, (5, 5, 6)
    cl = np.repeat(np.arange(3), sizes)
    lrs = []
    for q in range(groups):
        y, z = 8 * (q % 23), 8 * (q // 23)
        lrs += [LR.box_locreg((8 * c, y, z), (11, 7, 7), (8 * c + 3, y + 2, z + 2),
                              (8 * c + 6, y + 4, z + 4)) for c in cl]
    plan = W.Plan(W.Context(0.45, (32, 192, 192)), *to_abi(lrs))
    mask = np.abs(cl[:, None] - cl[None, :]) <= 1
    rows, cols = np.nonzero(mask)
    zin = torch.zeros(max(1, plan.info["in_coefs"]), dtype=torch.float64, device="cuda")
    W.sparse_overlap(plan, zin, zin, False, values=False)
    rng = np.random.default_rng(4400)
    R1, R2 = rng.standard_normal((m, m)), rng.standard_normal((m, m))
    S = (np.eye(m) + 0.1 / np.sqrt(m) * (R1 + R1.T)) * mask
    H = (np.diag(np.linspace(-1.0, 1.0, m)) + 0.5 / np.sqrt(m) * (R2 + R2.T)) * mask
    npl, delta, nocc = 30, 0.4, 0.5 * m
    K, mu, ebs, bnd = F.foe(S, H, mask, npl, delta, nocc)
    ktol, mtol = _tolerances(bnd, delta)
    print(f"case: FOE, {groups} groups of {m}", flush=True)
    kv, gmu, gebs = W.foe(plan, torch.tensor(np.tile(S[rows, cols], groups), device="cuda"),
                          torch.tensor(np.tile(H[rows, cols], groups), device="cuda"), npl, delta,
                          groups * nocc)
    got = kv.cpu().numpy().reshape(groups, -1)
    assert np.array_equal(got, np.broadcast_to(got[0], got.shape))
    assert np.max(np.abs(got[0] - K[rows, cols])) <= ktol * np.max(np.abs(K))
    assert abs(gmu - mu) <= mtol
    assert abs(gebs - groups * ebs) <= 1e-10 * groups * max(1.0, abs(ebs))
