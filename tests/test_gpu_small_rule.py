"""Which calls take the one-wavefront-per-row kernels: the choice follows the
rows, the beads, the model's shape and cutoffs and the lists' capacities, and
either choice gives the same bits as the other (the system inside a batch too
large for them).  The kernels of a call are read from the per-kernel timing:
the general ones alone have an angular force launch."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_small import gas
from test_gpu_triclinic import L, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

METAL = I.NepHyper(1, 5.0, 4.0, 4, 4, 8, 8, 4, False, 30)
LONG = I.NepHyper(1, 6.0, 5.0, 4, 4, 8, 8, 4, False, 30)
WATER = I.NepHyper(2, 6.0, 4.0, 4, 4, 8, 8, 4, False, 50)
FRAME = I.NepHyper(4, 6.0, 4.0, 8, 6, 8, 8, 4, False, 80)


def small_launch(L, torch, model, parts, P, caps):
    off = np.concatenate([[0], np.cumsum([p.shape[1] for p, _, _ in parts])]).astype(np.int32)
    offs = off if len(parts) > 1 else None
    pos = torch.tensor(np.concatenate([p for p, _, _ in parts], axis=1), dtype=torch.float64, device="cuda")
    typ = torch.tensor(np.concatenate([t for _, t, _ in parts]), dtype=torch.int32, device="cuda")
    box = np.stack([b for _, _, b in parts]) if offs is not None else parts[0][2]
    n = int(off[-1])
    nl = L.NeighborList(model, P, n, *caps, offsets=offs)
    ws = L.Workspace(model, P, n, offsets=offs)
    E = torch.zeros((len(parts), P), dtype=torch.float64, device="cuda")
    W = torch.zeros((len(parts), P, 9), dtype=torch.float64, device="cuda")
    F = torch.zeros((P, n, 3), dtype=torch.float32, device="cuda")
    if offs is None:
        E, W = E[0], W[0]
    nl.build(pos, box, typ)
    L.profile_enable(True)
    L.profile_read()
    ws.compute(nl, pos, box, typ, E, F, W)
    torch.cuda.synchronize()
    count = L.profile_read()
    L.profile_enable(False)
    assert nl.poll()[0] == 0 and ws.poll() == 0
    assert count["descriptor"][1] == 1 and count["force"][1] == 1
    first = off[1]
    one = (lambda x: x.reshape(len(parts), P, -1)[0].cpu().numpy())
    return count["force_ang"][1] == 0, one(E), one(W), F[:, :first].cpu().numpy()


@pytest.mark.parametrize("h,mlp,P,rows,caps,small", [
    (METAL, "fp32", 1, 8192, (60, 40), True), (METAL, "fp32", 1, 8193, (60, 40), False),
    (METAL, "fp32", 1, 12288, (60, 40), False), (METAL, "fp32", 4, 9000, (60, 40), False),
    (METAL, "fp32", 8, 12288, (60, 40), True), (METAL, "fp32", 8, 12296, (60, 40), False),
    (METAL, "fp32", 8, 6144, (22, 16), True), (METAL, "fp32", 8, 6152, (22, 16), False),   # lists of half the full length
    (LONG, "fp32", 1, 12288, (90, 50), True), (WATER, "fp32", 1, 12288, (90, 50), True),
    (WATER, "fp32", 1, 6144, (16, 16), True), (WATER, "fp32", 1, 6145, (16, 16), False),
    (LONG, "bf16_mfma", 16, 6144, (60, 40), True), (LONG, "bf16_mfma", 16, 6160, (60, 40), False),
    (FRAME, "fp32_mfma", 8, 6144, (30, 16), True), (FRAME, "fp32_mfma", 64, 6144, (30, 16), False),
    (FRAME, "fp32_mfma", 64, 3008, (24, 16), True), (FRAME, "fp32_mfma", 64, 3136, (24, 16), False)])
def test_rule(torch, L, tmpdir_session, h, mlp, P, rows, caps, small):  # noqa: F811
    n = rows // P
    edge = max((n / 0.004) ** (1 / 3), 2.2 * h.rc_radial)   # thin enough for every capacity above
    model = L.Model(write_model(tmpdir_session, "rule", I.random_model(h, np.random.default_rng(3), 0.004, 10.0)))
    model.set_mlp(L.MLP_MODES[mlp])
    box = np.diag([edge, edge * 1.01, edge * 1.03])
    pos, types = gas(n, box, h.n_species, P, 31)
    took, E, W, F = small_launch(L, torch, model, [(pos, types, box)], P, caps)
    assert took == small
    more = 13000 // P
    far = np.diag([(more / 0.004) ** (1 / 3)] * 3)
    fill = gas(more, far, h.n_species, P, 32)
    took, E2, W2, F2 = small_launch(L, torch, model, [(pos, types, box), (fill[0], fill[1], far)], P, caps)
    assert not took
    np.testing.assert_array_equal(F, F2)
    np.testing.assert_array_equal(E, E2)
    np.testing.assert_array_equal(W, W2)
    assert np.abs(F).max() > 0
