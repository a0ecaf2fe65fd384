"""A call repeated on the same state gives the same bits: nothing that a
kernel stores depends on when the instructions behind the store run.  The
model shapes whose adjoint rows are written wavefront-interleaved (parked
angular sums with a matrix-core or vector network, and B itself), over
enough workgroups to fill the chip."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_small import MODELS, SMALL_ROWS
from test_gpu_triclinic import L, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["teacher", "framework", "binary_mf", "metal4"])
def test_repeated_calls_same_bits(L, torch, tmpdir_session, name):  # noqa: F811
    h, mlp = MODELS[name]
    P, k, a = 32, 16, 3.0   # k^3 atoms, two (x 32 beads) per wavefront
    n = k ** 3
    rng = np.random.default_rng(7)
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3) * a
    pos = torch.tensor(g[None] + rng.normal(0.0, 0.08, (P, n, 3)), dtype=torch.float64, device="cuda")
    typ = torch.tensor(np.arange(n) % h.n_species, dtype=torch.int32, device="cuda")
    box = np.diag([k * a] * 3)
    model = L.Model(write_model(tmpdir_session, "rep_" + name,
                                I.random_model(h, np.random.default_rng(3), 1.0 / a ** 3, 10.0)))
    model.set_mlp(L.MLP_MODES[mlp])
    assert P * n > SMALL_ROWS
    nl = L.fitted_neighbor_list(model, pos, box, typ, 200, 120)
    ws = L.Workspace(model, P, n)
    E = torch.zeros(P, dtype=torch.float64, device="cuda")
    W = torch.zeros((P, 9), dtype=torch.float64, device="cuda")
    F = torch.zeros((P, n, 3), dtype=torch.float32, device="cuda")
    nl.build(pos, box, typ)
    ws.compute(nl, pos, box, typ, E, F, W)
    ref = (E.clone(), F.clone(), W.clone())
    assert bool(torch.isfinite(F).all())
    for _ in range(100):
        ws.compute(nl, pos, box, typ, E, F, W)
        for a_, b_ in zip((E, F, W), ref):
            assert torch.equal(a_, b_)
