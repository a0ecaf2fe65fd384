"""Packed positions of the force kernels on both sides of the rule that
chooses their form (fixed point up to 256 A edges, the fine grid beyond and
for general cells): smallest allowed and long cells, atoms in far periodic
images and on cell faces, against the oracle.  Bars as everywhere:
|dE|/N <= 1e-6 eV, max|dF| <= 1e-5 max|F|, max|dW| <= 1e-5 max|W|; the
per-bead neighbour sets bit for bit."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import configs
from test_gpu_nep import check_lists
from test_gpu_triclinic import E_TOL, F_TOL, W_TOL, L, evaluate, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def jittered(box, P, seed):
    """A jittered grid of atoms (two species), some of them displaced by whole edges, some on the faces."""
    rng = np.random.default_rng(seed)
    edges = np.diag(box)
    n = np.maximum(np.floor(edges / 3.3).astype(int), 1)
    grid = np.stack(np.meshgrid(*[np.arange(k) for k in n], indexing="ij"), -1).reshape(-1, 3)
    p0 = (grid + 0.5) / n * edges + rng.uniform(-0.5, 0.5, (grid.shape[0], 3))
    p0[::17, 0] = 0.0                                  # exactly on a face
    frac = p0 / edges
    frac += rng.integers(-3, 4, frac.shape)            # far images, every bead of an atom in the same one
    base = frac @ box
    types = (rng.random(len(base)) < 0.5).astype(np.int32)
    order = np.argsort(types, kind="stable")
    pos = base[order][None] + rng.normal(0.0, 0.05, (P,) + base.shape)
    return pos, types[order]


@pytest.mark.parametrize("edge,shear", [(12.3, 0.0), (64.0, 0.0), (256.0, 0.0), (256.5, 0.0), (300.0, 0.0),
                                        (256.0, 0.2)])
def test_position_forms(torch, L, orc, tmpdir_session, edge, shear):
    path = write_model(tmpdir_session, "positions", configs.WORKLOADS["rocksalt4096"].model())
    H = np.diag([edge, 13.1, 14.7])
    H[1, 0] = shear * 13.1
    P = 3
    pos, types = jittered(H, P, int(edge))
    box = H if shear else np.diag(H)
    got, nl, m = evaluate(torch, L, path, pos, types, box)
    tpos = torch.tensor(pos, dtype=torch.float64, device="cuda")
    check_lists(orc, nl.to_host(tpos, box), pos, box, m.rc_radial, m.rc_angular, types=types)
    M = orc.Model(path)
    for b in range(P):
        ref = M.config(pos[b], types, box)
        assert abs(got[0][b] - ref["E"]) / pos.shape[1] <= E_TOL
        assert np.abs(got[1][b] - ref["F"]).max() <= F_TOL * np.abs(ref["F"]).max()
        assert np.abs(got[2][b] - ref["W"]).max() <= W_TOL * np.abs(ref["W"]).max()
