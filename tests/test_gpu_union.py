"""Union lists of the force path against the oracle: lane groups from one
bead to a whole wavefront (shell candidates tested 64 down to one at a time),
candidate rows shorter and longer than a wavefront in the list, its shell and
the reverse slots, with the centroid records of orthorhombic cells and the
FP64 centroids of general ones.  Bars: |dE|/N <= 1e-6 eV, max|dF| <= 1e-5
max|F|, max|dW| <= 1e-5 max|W|."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_triclinic import E_TOL, F_TOL, W_TOL, L, evaluate, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,spread,pitch,rc,shear", [
    (1, 0.0, 2.2, (6.0, 5.2), 0.0), (2, 0.05, 2.2, (6.0, 5.2), 0.0), (3, 0.3, 2.6, (6.0, 4.0), 0.0),
    (5, 0.6, 2.2, (6.0, 5.2), 0.0), (33, 0.25, 2.6, (6.0, 5.0), 0.0), (64, 0.5, 2.9, (6.0, 4.0), 0.0),
    (5, 0.6, 2.2, (6.0, 5.2), 0.15), (33, 0.25, 2.6, (6.0, 5.0), 0.15)])
def test_union_against_oracle(torch, L, orc, tmpdir_session, P, spread, pitch, rc, shear):  # noqa: F811
    h = I.NepHyper(2, rc[0], rc[1], 4, 4, 8, 8, 4, False, 20)
    k = 7
    edge = k * pitch
    rng = np.random.default_rng(P)
    grid = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)
    H = np.diag([edge, edge, edge])
    H[1, 0] = shear * edge
    base = ((grid + 0.5 + rng.uniform(-0.1, 0.1, grid.shape)) / k) @ H
    types = (rng.random(len(base)) < 0.5).astype(np.int32)
    order = np.argsort(types, kind="stable")
    pos = base[order][None] + rng.uniform(-spread, spread, (P,) + base.shape)
    types = types[order]
    path = write_model(tmpdir_session, "union", I.random_model(h, np.random.default_rng(5), 1.0 / pitch ** 3, 10.0))
    box = H if shear else np.diag(H)
    got = evaluate(torch, L, path, pos, types, box)[0]
    M = orc.Model(path)
    for b in sorted({0, P // 2, P - 1}):
        ref = M.config(pos[b], types, box)
        assert abs(got[0][b] - ref["E"]) / pos.shape[1] <= E_TOL
        assert np.abs(got[1][b] - ref["F"]).max() <= F_TOL * np.abs(ref["F"]).max()
        assert np.abs(got[2][b] - ref["W"]).max() <= W_TOL * np.abs(ref["W"]).max()
