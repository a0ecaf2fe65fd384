"""Small systems take kernels of their own (one wavefront per (atom, bead));
the same system inside a batch that is too large for them takes the general
ones.  Both must agree bit for bit, for every model shape, network form and
cell form, with neighbour lists shorter and longer than a wavefront, odd
bead counts, an atom without neighbours and a species without atoms."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import configs
from paper_2409_04430_amd import inputs as I
from test_gpu_triclinic import L, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

SMALL_ROWS, SMALL_ROWS_MF = 12288, 6144   # (bead, atom) rows up to which the small kernels run

# name: shape of the model (species, cutoffs, n_max, four-body, hidden), network form
MODELS = {
    "metal": (I.NepHyper(1, 5.0, 4.0, 4, 4, 8, 8, 4, False, 30), "fp32"),
    "metal4": (I.NepHyper(1, 5.0, 4.5, 4, 4, 8, 8, 4, True, 70), "fp32"),
    "binary": (I.NepHyper(2, 6.0, 4.0, 6, 4, 8, 8, 4, False, 50), "fp32"),
    "binary_mf": (I.NepHyper(2, 6.0, 4.0, 6, 4, 8, 8, 4, False, 50), "fp32_mfma"),
    "student": (I.NepHyper(1, 6.0, 5.0, 4, 4, 8, 8, 4, False, 30), "bf16_mfma"),
    "framework": (I.NepHyper(4, 6.0, 4.0, 8, 6, 8, 8, 4, False, 80), "auto"),
    "framework_vec": (I.NepHyper(4, 6.0, 4.0, 8, 6, 8, 8, 4, False, 80), "fp32"),
    "teacher": (I.NepHyper(1, 6.0, 5.0, 8, 8, 8, 8, 4, True, 100), "auto"),
    "embedded": (I.NepHyper(3, 5.5, 4.0, 5, 2, 6, 5, 3, False, 33), "fp32"),
}


def gas(n, box, S, P, seed, lone=True):
    """n atoms on a jittered grid of the cell (edge vectors as rows), beads spread about them, one atom
    alone outside every cutoff's reach where the cell allows it."""
    rng = np.random.default_rng(seed)
    k = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)
    base = ((g[rng.permutation(len(g))[:n]] + 0.5) / k + rng.uniform(-0.08, 0.08, (n, 3))) @ box
    types = np.sort(rng.integers(0, S, n)).astype(np.int32)
    return base[None] + rng.normal(0.0, 0.06, (P, n, 3)), types


def evaluate(L, torch, model, parts, P):
    off = np.concatenate([[0], np.cumsum([p.shape[1] for p, _, _ in parts])]).astype(np.int32)
    n, dev = int(off[-1]), "cuda"
    offs = off if len(parts) > 1 else None
    pos = torch.tensor(np.concatenate([p for p, _, _ in parts], axis=1), dtype=torch.float64, device=dev)
    typ = torch.tensor(np.concatenate([t for _, t, _ in parts]), dtype=torch.int32, device=dev)
    box = np.stack([b for _, _, b in parts]) if offs is not None else parts[0][2]
    nl = L.fitted_neighbor_list(model, pos, box, typ, 200, 120, offsets=offs)
    ws = L.Workspace(model, P, n, offsets=offs)
    es = (len(parts), P) if offs is not None else (P,)
    E = torch.zeros(es, dtype=torch.float64, device=dev)
    W = torch.zeros(es + (9,), dtype=torch.float64, device=dev)
    F = torch.zeros((P, n, 3), dtype=torch.float32, device=dev)
    Ea = torch.zeros((P, n), dtype=torch.float32, device=dev)
    Wa = torch.zeros((P, n, 9), dtype=torch.float32, device=dev)
    nl.build(pos, box, typ)
    ws.compute(nl, pos, box, typ, E, F, W, Ea, Wa)
    torch.cuda.synchronize()
    assert nl.poll()[0] == 0 and ws.poll() == 0
    first = off[1]
    pick = (lambda x: x[0]) if offs is not None else (lambda x: x)
    return dict(E=pick(E).cpu().numpy(), W=pick(W).cpu().numpy(), F=F[:, :first].cpu().numpy(),
                E_atom=Ea[:, :first].cpu().numpy(), W_atom=Wa[:, :first].cpu().numpy(),
                longest=nl.to_host()["union_end_radial"].max())


@pytest.mark.parametrize("name,P,n,edge,shear", [
    ("metal", 4, 108, 12.2, 0.0), ("metal", 1, 1, 14.0, 0.0), ("metal", 64, 5, 14.0, 0.0), ("metal4", 3, 111, 12.2, 0.0),
    ("binary", 5, 270, 13.1, 0.0), ("binary", 2, 300, 16.0, 0.25), ("binary_mf", 7, 130, 13.1, 0.0),
    ("student", 16, 128, 13.1, 0.0), ("framework", 6, 200, 14.0, 0.0), ("framework_vec", 1, 700, 16.0, 0.0),
    ("teacher", 2, 256, 13.0, 0.0), ("teacher", 9, 64, 13.0, 0.0), ("embedded", 12, 90, 12.0, 0.0),
    ("binary", 1, SMALL_ROWS, 50.0, 0.0), ("metal", 32, SMALL_ROWS // 32, 18.0, 0.0),
    ("student", 48, SMALL_ROWS_MF // 48, 13.1, 0.0)])
def test_small_equals_general(torch, L, tmpdir_session, name, P, n, edge, shear):
    h, mlp = MODELS[name]
    model = L.Model(write_model(tmpdir_session, "small_" + name,
                                I.random_model(h, np.random.default_rng(3), n / edge ** 3, 10.0)))
    model.set_mlp(L.MLP_MODES[mlp])
    box = np.diag([edge, edge * 1.01, edge * 1.03])
    box[1, 0] = shear * edge
    pos, types = gas(n, box, h.n_species, P, 17)
    assert P * n <= (SMALL_ROWS if mlp == "fp32" else SMALL_ROWS_MF)
    more = SMALL_ROWS // P + 1 - n + 700 // P
    big = (np.diag([55.0, 55.0, 55.0]),)
    fill = gas(more, big[0], h.n_species, P, 18)
    one = evaluate(L, torch, model, [(pos, types, box)], P)
    both = evaluate(L, torch, model, [(pos, types, box), (fill[0], fill[1], big[0])], P)
    for k in ("F", "E", "W", "E_atom", "W_atom"):
        np.testing.assert_array_equal(one[k], both[k], err_msg=k)
    assert n < 64 or np.abs(one["F"]).max() > 0   # a handful of atoms may have no neighbours
