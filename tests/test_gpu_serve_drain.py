"""auv_session_drain returns only when every request submitted before it is done,
also while the worker is between taking a request from its queue and having
launched it (the session is drained at once after each submit, many times)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_nothing_runs_after_drain():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    grids = [ag.make_desc(0.0, 0.0, 2.0, 2.0, 128, 128)]
    desc = ag.session_desc(grids, radius=6.0, max_request=4000, slots=4, z_ref=[-500.0])
    fixed, per = ag.auv_session_budget(desc)
    arena = torch.empty(fixed + per, dtype=torch.uint8, device="cuda")
    session = ag.Session(desc, arena)
    rng = np.random.default_rng(1)
    x, y = rng.uniform(0.0, 256.0, 2000), rng.uniform(0.0, 256.0, 2000)
    z = rng.normal(-500.0, 1.0, 2000)
    states = []
    for _ in range(1500):
        ticket = session.submit(0, x, y, z)
        session.drain()
        states.append(session.poll(ticket).state)
    session.close()
    assert all(s == ag.AUV_T_DONE for s in states)
