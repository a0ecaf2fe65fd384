"""Own angular sums in two parts: a system whose rows fit one lane per SIMD
lane is summed by two lanes per row on its own and by one lane, part after
part, inside a larger batch; a larger system, more than 32 lanes per atom and
wide angular sets are summed as a whole.  Alone and first in a batch every
form gives the same bits; sizes on both sides of each rule."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_small import MODELS, SMALL_ROWS, evaluate, gas
from test_gpu_triclinic import L, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

PART_ROWS = 65536   # rows (atom, bead) of a system up to which its sums are taken in parts


@pytest.mark.parametrize("name,P,n,shear", [
    ("metal", 32, PART_ROWS // 32, 0.0), ("metal", 32, PART_ROWS // 32 + 1, 0.0),
    ("metal4", 1, SMALL_ROWS + 1, 0.0), ("binary", 20, PART_ROWS // 32, 0.0), ("binary", 20, 3000, 0.2),
    ("binary_mf", 5, 2501, 0.2), ("student", 16, 4096, 0.0), ("metal", 33, 400, 0.0), ("framework", 32, 500, 0.0)])
def test_alone_equals_batch(torch, L, tmpdir_session, name, P, n, shear):  # noqa: F811
    h, mlp = MODELS[name]
    edge = (n * 14.0) ** (1 / 3)
    model = L.Model(write_model(tmpdir_session, "parts_" + name, I.random_model(h, np.random.default_rng(3), 1 / 14.0, 10.0)))
    model.set_mlp(L.MLP_MODES[mlp])
    box = np.diag([edge, edge * 1.01, edge * 1.03])
    box[1, 0] = shear * edge
    pos, types = gas(n, box, h.n_species, P, 21)
    more = PART_ROWS // P + 500   # takes the launch past two lanes per row, itself summed as a whole
    far = np.diag([(more * 14.0) ** (1 / 3)] * 3)
    fill = gas(more, far, h.n_species, P, 22)
    tiny = np.diag([15.0, 15.0, 15.0])
    last = gas(9, tiny, h.n_species, P, 23)
    assert P * n > SMALL_ROWS
    one = evaluate(L, torch, model, [(pos, types, box)], P)
    both = evaluate(L, torch, model, [(pos, types, box), (fill[0], fill[1], far), (last[0], last[1], tiny)], P)
    for k in ("F", "E", "W", "E_atom", "W_atom"):
        np.testing.assert_array_equal(one[k], both[k], err_msg=k)
    assert np.abs(one["F"]).max() > 0
