"""Graphs launched in a row: no more than the schedule has left, and nothing
planned by a run that came before.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rcp():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2608_12235_amd as m
    m.lib()
    return m


def _launches(p):
    return p.stats()["graph_launches"]


def test_short_calls_after_a_long_run_launch_little(rcp, orc):
    # a settling run has list builds hundreds of iterations apart; a step, a
    # few steps, and a new run of a few steps after it take a graph each
    n, L = 300, 7.0
    d = 0.5 + 0.1 * np.arange(n) / n
    x = orc.rsa(d, L, 0.5, 5)
    long_run = rcp.schedule_from_rungs([(1e-4, 1e-3, 1e-4, 1.0, 4000)], tol=-1.0)
    p = rcp.Packing(d, L, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.1))
    p.set_state(x, 1.2)
    p.inflate_run(long_run)
    assert p.stats()["rebuilds"] >= 3      # (an interval is known)
    for steps in (1, 3, 8):
        before = _launches(p)
        p.adam_step(1e-5, 1e-5, 1e-6, steps)
        assert _launches(p) - before == 1, steps
    # from a new state: the list is built at its first iteration, and then
    # nothing is known but that the first graph may be a whole one
    p.set_state(x, 1.2)
    before = _launches(p)
    p.run_start(rcp.schedule_from_rungs([(1e-2, 5e-2, 5e-3, 1.0, 1 << 30)], tol=-1.0))
    p.run_continue(40)
    first = _launches(p) - before
    q = rcp.Packing(d, L, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.1))
    q.set_state(x, 1.2)
    q.run_start(rcp.schedule_from_rungs([(1e-2, 5e-2, 5e-3, 1.0, 1 << 30)], tol=-1.0))
    q.run_continue(40)
    assert first == _launches(q)
    assert np.array_equal(p.get_state()[0], q.get_state()[0])
    p.close()
    q.close()
