"""Pair histograms on both sides of the lane count that changes how many
threads share a list (131,072 lanes, the beads of an atom in the next power
of two of them), with short lists and with lists of many batches, several
species and both cell forms: every count as the oracle's, accumulating twice
doubles it."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import inputs as I
from test_gpu_rdf import L, gpu_hist, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,P,n,spacing,shear", [
    (2, 64, 2048, 2.2, 0.0), (2, 64, 2049, 2.2, 0.0), (4, 48, 2100, 4.2, 0.0), (3, 33, 2300, 2.8, 0.2),
    (1, 64, 2048, 4.2, 0.0)])
def test_counts(torch, L, orc, tmpdir_session, S, P, n, spacing, shear):  # noqa: F811
    h = I.NepHyper(S, 5.0, 4.0, 4, 4, 8, 8, 4, False, 10)
    path = write_model(tmpdir_session, "rdf_lanes", I.random_model(h, np.random.default_rng(3), spacing ** -3, 10.0))
    rng = np.random.default_rng(n + P)
    k = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)
    H = np.diag([k * spacing] * 3)
    H[1, 0] = shear * H[1, 1]
    base = ((g[rng.permutation(len(g))[:n]] + 0.5 + rng.uniform(-0.2, 0.2, (n, 3))) / k) @ H
    types = rng.integers(0, S, n).astype(np.int32)
    pos = base[None] + rng.normal(0.0, 0.05, (P, n, 3))
    box = H if shear else np.diag(H).copy()
    got, _, _ = gpu_hist(torch, L, path, pos, types, box, 4.9, 77, repeat=2, caps=(200, 120))
    ref = orc.rdf_counts(pos, types, box, 4.9, 77, S)
    assert ref.sum() > 0
    np.testing.assert_array_equal(got, 2 * ref)
