"""The gradient kernels at the sizes where their loops change: neighbour
lists of up to 32, up to 64 and more entries, several species with blocks of
their own, hidden layers across more than one tile, row counts off the chunk
sizes.  Per parameter block, the derivative along a random direction against
central differences of the FP64 oracle loss; bar 2e-3 of the largest of them,
as for the single entries in test_gpu_train.py."""
import copy

import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_small import gas
from test_gpu_train import L, LAM, gpu_grad, oracle_loss, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,n,edge,P", [
    (I.NepHyper(4, 6.3, 6.2, 8, 6, 8, 8, 4, False, 81), 215, 13.2, 1),    # angular lists past 64 entries
    (I.NepHyper(3, 5.5, 4.6, 8, 6, 8, 8, 4, False, 33), 125, 12.0, 3),    # blocks within the second stage
    (I.NepHyper(2, 6.0, 3.6, 6, 4, 8, 8, 4, False, 130), 100, 12.6, 2),   # a single stage, five hidden tiles
    (I.NepHyper(1, 6.0, 5.0, 4, 4, 8, 8, 4, False, 1), 17, 13.0, 5)])     # one hidden unit, few rows
def test_directional_derivatives(torch, L, orc, tmpdir_session, h, n, edge, P):
    rng = np.random.default_rng(11)
    student = I.random_model(h, rng, n / edge ** 3, 5.0)
    path = write_model(tmpdir_session, "rows", student)
    box = np.array([edge, edge * 1.02, edge * 1.05])
    pos, types = gas(n, np.diag(box), h.n_species, P, 4)
    model = orc.Model(path).beads(pos, types, box)
    ref = {k: np.asarray(model[k]) for k in ("E", "F", "W")}
    ref["E"] = ref["E"] + rng.normal(0.0, 0.1 * n, P)
    ref["F"] = ref["F"] + rng.normal(0.0, 0.3, (P, n, 3))
    ref["W"] = ref["W"] + rng.normal(0.0, 0.1 * n, ref["W"].shape)
    m, nl, ws, tr, tpos, ttyp, refs = gpu_grad(torch, L, path, ref, pos, types, box)
    nl.build(tpos, box, ttyp)
    tr.zero()
    tr.accumulate(nl, ws, tpos, box, ttyp, *refs, LAM)
    torch.cuda.synchronize()
    g, loss = tr.grad.cpu().numpy().astype(np.float64), tr.loss.cpu().numpy()
    L0 = oracle_loss(orc, tmpdir_session, student, ref, pos, types, box)
    assert abs(loss[0] - L0) <= 1e-4 * L0
    assert abs(loss[0] - loss[1:].sum()) <= 1e-12 * loss[0]
    got, fd = [], []
    for name in ("W0", "b0", "w1", "c_radial", "c_angular"):
        d = rng.normal(size=student[name].shape)
        d /= np.linalg.norm(d)
        vals = []
        for sign in (1, -1):
            mm = copy.deepcopy(student)
            mm[name] = student[name] + sign * 1e-4 * d
            vals.append(oracle_loss(orc, tmpdir_session, mm, ref, pos, types, box))
        fd.append((vals[0] - vals[1]) / 2e-4)
        got.append(g[tr.offsets[name]:tr.offsets[name] + d.size] @ d.ravel())
    got, fd = np.array(got), np.array(fd)
    print(np.c_[got, fd], flush=True)
    assert np.all(np.abs(got - fd) <= 2e-3 * np.abs(fd).max() + 1e-7)
