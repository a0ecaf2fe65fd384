"""Batches of systems with different forms of packed positions (fixed point,
the fine grid of a long orthorhombic cell, the fine grid of a general cell):
a launch carries the code of one form or of all, and every system keeps the
bits that it has on its own, in the small-system kernels and the general
ones."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_small import SMALL_ROWS, evaluate
from test_gpu_triclinic import L, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def lattice(edges, shear, S, P, seed):
    rng = np.random.default_rng(seed)
    H = np.diag(np.asarray(edges, float))
    H[1, 0] = shear * edges[1]
    k = np.round(np.asarray(edges) / 2.6).astype(int)
    g = np.stack(np.meshgrid(*[np.arange(n) for n in k], indexing="ij"), -1).reshape(-1, 3)
    base = ((g + 0.5) / k + rng.uniform(-0.03, 0.03, g.shape) / k) @ H
    types = np.sort(rng.integers(0, S, len(g))).astype(np.int32)
    return base[None] + rng.normal(0.0, 0.06, (P,) + base.shape), types, H


@pytest.mark.parametrize("P", [1, 16])
@pytest.mark.parametrize("forms", [("fixed", "grid", "general"), ("grid", "long"), ("general", "fixed"), ("fixed", "edge")])
def test_forms_beside_each_other(torch, L, tmpdir_session, forms, P):  # noqa: F811
    h = I.NepHyper(2, 6.0, 4.5, 4, 4, 8, 8, 4, False, 30)
    model = L.Model(write_model(tmpdir_session, "forms", I.random_model(h, np.random.default_rng(3), 1 / 17.6, 10.0)))
    cells = {"fixed": ((24.0, 26.1, 23.7), 0.0), "grid": ((210.0, 13.1, 14.3), 0.0), "general": ((24.0, 26.1, 23.7), 0.2),
             "long": ((14.1, 13.3, 300.0), 0.0), "edge": ((200.0, 13.5, 14.0), 0.0)}
    parts = [lattice(*cells[f], h.n_species, P, 5 + k) for k, f in enumerate(forms)]
    rows = P * sum(p.shape[1] for p, _, _ in parts)
    assert (rows > SMALL_ROWS) == (P > 1)
    for k in range(len(parts)):
        one = evaluate(L, torch, model, [parts[k]], P)
        both = evaluate(L, torch, model, parts[k:] + parts[:k], P)
        for key in ("F", "E", "W", "E_atom", "W_atom"):
            np.testing.assert_array_equal(one[key], both[key], err_msg=f"{forms[k]} {key}")
        assert np.abs(one["F"]).max() > 0
