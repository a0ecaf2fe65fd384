"""Energies and virials of a student run's steps whose sums are left to the
integrator launch: after an unjudged step on the student and after one on
the teacher (fallen back), E and W equal bit for bit those of a plain
evaluation of the same positions, in the small-system form of the pending
sums and in the general one."""
import numpy as np
import pytest

from conftest import write_model
from paper_2409_04430_amd import configs
from paper_2409_04430_amd import inputs as I
from test_gpu_triclinic import L, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,ncell", [(4, 4), (32, 5)])   # 1,024 rows and 16,000, on both sides of every row limit
def test_sums_after_unjudged_steps(torch, L, tmpdir_session, P, ncell):  # noqa: F811
    from paper_2409_04430_amd.student import StudentPimd
    w = configs.WORKLOADS["fcc32000"]
    tpath = write_model(tmpdir_session, "sums_teacher", w.model())
    spath = write_model(tmpdir_session, "sums_student", w.model(student=True))
    p0, t, b = I.fcc(ncell, 4.05)
    system = I.make_system(p0, t, b, w.species_masses, P, 500.0, 0.05, np.random.default_rng(31))
    st = StudentPimd(tpath, spath, system, dt=w.dt, T=500.0, mode="trpmd", seed=6, judge_every=3, threshold=1e9,
                     check_every=0)
    e = st.eng

    def checked_step(ws):
        E, F, W = torch.zeros_like(e.E), torch.zeros_like(e.F), torch.zeros_like(e.W)
        e.nl.build(e.pos, e.box, e.types)
        ws.compute(e.nl, e.pos, e.box, e.types, E, F, W)
        for x in (e.E, e.W, e.F):
            x.fill_(float("nan"))
        st.step()
        torch.cuda.synchronize()
        assert torch.equal(e.F, F) and torch.equal(e.E, E) and torch.equal(e.W, W)
        assert float(E.abs().min()) > 0.0 and float(W.abs().max()) > 0.0

    st.run(1)                        # step 0, judged
    checked_step(e.ws)               # steps 1 and 2 on the student
    checked_step(e.ws)
    assert st.on_student and [s for s, _ in st.history] == [0]
    st.threshold = -1.0
    st.run(1)                        # step 3, judged: falls back
    assert not st.on_student and st.fallback_step == 3
    checked_step(st.tws)
    st.run(1)
    checked_step(st.tws)             # step 6 would be judged on the student
    st.check()
