"""Rounding of the pair vectors of the force kernels.  Two atoms beyond the
angular cutoff have the radial pair term w r alone, so that F_a = w d_a (one
FP32 rounding) and W_atom_aa = -1/2 d_a F_a (another): d_a is read back from
-2 W_atom_aa / F_a.  The error of the vector is bounded by one FP32 rounding
of each component and the resolution of the stored positions: at most one
quantum L / 2^32 in fixed point (orthorhombic edges up to 200 A, and on both
sides of that rule), on the fine grid beyond that rule two offsets below 1 A
and their difference (3/2 of 2^-24) and the FP32 grid step (2^-24 of the
component)."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_triclinic import L, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

FIXED_MAX_EDGE = 200.0


def half_ulp(d):
    return 2.0 ** (np.floor(np.log2(np.abs(d))) - 24)


# 64 systems take the small-system kernels, 200 the general ones
@pytest.mark.parametrize("nsys,lo,hi", [(64, 10.2, 60.0), (200, 10.2, 199.0), (200, 200.0, 200.0), (200, 200.5, 300.0),
                                        (200, 150.0, 260.0)])
def test_one_rounding(torch, L, tmpdir_session, nsys, lo, hi):  # noqa: F811
    h = I.NepHyper(1, 5.0, 2.0, 4, 4, 8, 8, 4, False, 10)
    model = L.Model(write_model(tmpdir_session, "pairs", I.random_model(h, np.random.default_rng(2), 0.05, 10.0)))
    rng = np.random.default_rng(nsys + int(lo))
    P, n = 64, 2 * nsys
    edges = rng.uniform(lo, hi, (nsys, 3))
    u = rng.normal(size=(nsys, P, 3))
    d = u / np.linalg.norm(u, axis=-1, keepdims=True) * rng.uniform(2.2, 4.5, (nsys, P, 1))
    a = rng.uniform(-1.0, 2.0, (nsys, 1, 3)) * edges[:, None] + rng.normal(0.0, 0.1, (nsys, P, 3))
    pos = np.stack([a, a + d], axis=2).transpose(1, 0, 2, 3).reshape(P, n, 3)   # [bead][system, atom]
    d = (pos[:, 1::2] - pos[:, 0::2])                                            # as stored
    box = np.stack([np.diag(e) for e in edges])
    off = np.arange(0, n + 1, 2, dtype=np.int32)
    tpos = torch.tensor(pos, dtype=torch.float64, device="cuda")
    typ = torch.zeros(n, dtype=torch.int32, device="cuda")
    nl = L.fitted_neighbor_list(model, tpos, box, typ, 8, 8, offsets=off)
    ws = L.Workspace(model, P, n, offsets=off)
    E = torch.zeros((nsys, P), dtype=torch.float64, device="cuda")
    W = torch.zeros((nsys, P, 9), dtype=torch.float64, device="cuda")
    F = torch.zeros((P, n, 3), dtype=torch.float32, device="cuda")
    Ea = torch.zeros((P, n), dtype=torch.float32, device="cuda")
    Wa = torch.zeros((P, n, 9), dtype=torch.float32, device="cuda")
    nl.build(tpos, box, typ)
    ws.compute(nl, tpos, box, typ, E, F, W, Ea, Wa)
    torch.cuda.synchronize()
    assert nl.poll()[0] == 0 and ws.poll() == 0
    f = F[:, 0::2].cpu().numpy().astype(np.float64)
    w = Wa[:, 0::2].cpu().numpy().astype(np.float64)[..., [0, 4, 8]]
    ok = np.abs(f) > 1e-30
    assert ok.mean() > 0.99
    got = np.where(ok, -2.0 * w / np.where(ok, f, 1.0), d)
    fixed = (edges.max(1) <= FIXED_MAX_EDGE)[None, :, None]
    step = np.where(fixed, edges[None] * 2.0 ** -32 * 1.001, 1.5 * 2.0 ** -24 + 2.0 ** -24 * np.abs(d))
    bar = half_ulp(np.abs(d) + step) + 2.0 ** -24 * np.abs(d) + step
    err = np.abs(got - d)
    print("rms %.3e largest %.3e of the bar %.3f" % (np.sqrt((err ** 2).mean()), err.max(), (err / bar).max()), flush=True)
    assert np.all(err <= bar)
