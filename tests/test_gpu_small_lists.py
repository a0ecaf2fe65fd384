"""The one-wavefront-per-row kernels on lists with holes: an atom without
neighbours, species (first, middle, last) without atoms, lists on both sides
of a wavefront's 64 entries.  Forces: bit for bit those of the general
kernels, and within the usual bars of the oracle (|dE|/N <= 1e-6 eV, max|dF|
<= 1e-5 max|F|, max|dW| <= 1e-5 max|W|).  Training rows: directional
derivatives per parameter block against central differences of the FP64
oracle loss, bar 2e-3 of the largest."""
import copy

import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_small import gas
from test_gpu_small_rule import small_launch
from test_gpu_train import LAM, gpu_grad, oracle_loss
from test_gpu_triclinic import E_TOL, F_TOL, W_TOL, L, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

# name: model, network form, species present, atoms, edge of the cell they fill, beads, longest list past 64
CASES = {
    "first_absent": (I.NepHyper(2, 6.0, 4.0, 6, 4, 8, 8, 4, False, 50), "fp32", (1,), 190, 12.4, 3, True),
    "last_absent": (I.NepHyper(2, 6.0, 4.0, 4, 4, 8, 8, 4, False, 50), "fp32", (0,), 60, 12.4, 5, False),
    "middle_absent": (I.NepHyper(3, 5.5, 4.6, 4, 4, 8, 8, 4, False, 33), "fp32", (0, 2), 200, 12.0, 2, True),
    "two_absent": (I.NepHyper(4, 6.0, 4.0, 8, 6, 8, 8, 4, False, 80), "fp32_mfma", (1, 2), 200, 12.4, 4, True),
    "ends_absent": (I.NepHyper(4, 6.0, 4.0, 8, 6, 8, 8, 4, False, 40), "fp32", (1, 3), 50, 12.4, 7, False),
    "four_body": (I.NepHyper(1, 6.0, 5.0, 8, 8, 8, 8, 4, True, 30), "fp32_mfma", (0,), 170, 12.4, 3, True),
}


def build(name, seed):
    """The case's atoms in one corner of a longer cell, and one more atom alone in the vacuum of it."""
    h, mlp, present, n, edge, P, past = CASES[name]
    corner = np.diag([edge, edge * 1.02, edge * 1.04])
    rng = np.random.default_rng(seed)
    m = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    base = ((g[np.sort(rng.permutation(len(g))[:n])] + 0.5 + rng.uniform(-0.15, 0.15, (n, 3))) / m) @ corner
    pos = base[None] + rng.normal(0.0, 0.06, (P, n, 3))
    types = np.sort(np.asarray(present)[rng.integers(0, len(present), n)])
    types[0], types[-1] = present[0], present[-1]
    box = corner + np.diag([2.5 * h.rc_radial, 0.0, 0.0])
    alone = np.array([edge + 1.25 * h.rc_radial, 0.5 * edge, 0.5 * edge]) + rng.normal(0.0, 0.06, (P, 1, 3))
    k = n // 2   # the lone atom within the order of its species
    pos = np.concatenate([pos[:, :k], alone, pos[:, k:]], axis=1)
    types = np.concatenate([types[:k], types[k:k + 1], types[k:]]).astype(np.int32)
    return pos, types, box, k


@pytest.mark.parametrize("name", sorted(CASES))
def test_forces(torch, L, orc, tmpdir_session, name):  # noqa: F811
    h, mlp, present, n, edge, P, past = CASES[name]
    pos, types, box, lone = build(name, 41)
    assert set(types.tolist()) == set(present) and len(present) <= h.n_species
    path = write_model(tmpdir_session, "lists_" + name, I.random_model(h, np.random.default_rng(3), n / edge ** 3, 10.0))
    model = L.Model(path)
    model.set_mlp(L.MLP_MODES[mlp])
    tpos = torch.tensor(pos, dtype=torch.float64, device="cuda")
    typ = torch.tensor(types, device="cuda")
    nl = L.fitted_neighbor_list(model, tpos, box, typ, 200, 120)
    nl.build(tpos, box, typ)
    longest = nl.to_host()["union_end_radial"].max(axis=1)
    assert longest[lone] == 0 and (longest.max() > 64) == past
    took, E, W, F = small_launch(L, torch, model, [(pos, types, box)], P, (200, 120))
    assert took
    more = 13000 // P
    far = np.diag([(more / 0.02) ** (1 / 3)] * 3)
    fill = gas(more, far, h.n_species, P, 42)
    took, E2, W2, F2 = small_launch(L, torch, model, [(pos, types, box), (fill[0], fill[1], far)], P, (200, 120))
    assert not took
    np.testing.assert_array_equal(F, F2)
    np.testing.assert_array_equal(E, E2)
    np.testing.assert_array_equal(W, W2)
    assert np.all(F[:, lone] == 0.0)
    M = orc.Model(path)
    for b in range(P):
        ref = M.config(pos[b], types, np.diag(box).copy())
        assert abs(E[b, 0] - ref["E"]) / len(types) <= E_TOL
        assert np.abs(F[b] - ref["F"]).max() <= F_TOL * np.abs(ref["F"]).max()
        assert np.abs(W[b].reshape(3, 3) - np.reshape(ref["W"], (3, 3))).max() <= W_TOL * np.abs(ref["W"]).max()


@pytest.mark.parametrize("name", [n for n in sorted(CASES) if not CASES[n][0].four_body])
def test_training_rows(torch, L, orc, tmpdir_session, name):  # noqa: F811
    h, _, present, n, edge, P, _ = CASES[name]
    pos, types, cell, lone = build(name, 51)
    box = np.diag(cell).copy()
    rng = np.random.default_rng(12)
    student = I.random_model(h, rng, n / edge ** 3, 5.0)
    path = write_model(tmpdir_session, "lists_rows", student)
    out = orc.Model(path).beads(pos, types, box)
    ref = {k: np.asarray(out[k]) for k in ("E", "F", "W")}
    ref["E"] = ref["E"] + rng.normal(0.0, 0.1 * n, P)
    ref["F"] = ref["F"] + rng.normal(0.0, 0.3, pos.shape)
    ref["W"] = ref["W"] + rng.normal(0.0, 0.1 * n, ref["W"].shape)
    m, nl, ws, tr, tpos, ttyp, refs = gpu_grad(torch, L, path, ref, pos, types, box)
    nl.build(tpos, box, ttyp)
    tr.zero()
    tr.accumulate(nl, ws, tpos, box, ttyp, *refs, LAM)
    torch.cuda.synchronize()
    g = tr.grad.cpu().numpy().astype(np.float64)
    L0 = oracle_loss(orc, tmpdir_session, student, ref, pos, types, box)
    assert abs(tr.loss.cpu().numpy()[0] - L0) <= 1e-4 * L0
    absent = [s for s in range(h.n_species) if s not in present]
    got, fd = [], []
    for key in ("W0", "b0", "w1", "c_radial", "c_angular"):
        lo = tr.offsets[key]
        block = g[lo:lo + student[key].size].reshape(student[key].shape)
        for s in absent:   # parameters of species without atoms: exactly no gradient, as centre and as neighbour
            assert np.all(block[s] == 0.0), key
            if key in ("c_radial", "c_angular"):
                assert np.all(block[:, s] == 0.0), key
        d = rng.normal(size=student[key].shape)
        d /= np.linalg.norm(d)
        vals = []
        for sign in (1, -1):
            mm = copy.deepcopy(student)
            mm[key] = student[key] + sign * 1e-4 * d
            vals.append(oracle_loss(orc, tmpdir_session, mm, ref, pos, types, box))
        fd.append((vals[0] - vals[1]) / 2e-4)
        got.append(float(block.ravel() @ d.ravel()))
    got, fd = np.array(got), np.array(fd)
    print(np.c_[got, fd], flush=True)
    assert np.all(np.abs(got - fd) <= 2e-3 * np.abs(fd).max() + 1e-7)
