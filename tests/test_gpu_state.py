"""Positions handed in from host and device memory: checked and wrapped as
documented, the optimiser at its start, a refused state without a trace."""
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


@pytest.mark.parametrize("walls", [0, 1, 5])
@pytest.mark.parametrize("n", [1, 85, 256, 257, 1500])
def test_host_positions_are_checked_and_wrapped(rcp, n, walls):
    L = 7.3
    rng = np.random.default_rng(n)
    p = rcp.Packing(0.05 + 0.05 * rng.random(n), L, 1.0, 0, init="none",
                    boundary=(walls, 0) if walls else None)
    x = rng.uniform(-L, 2 * L, (n, 3))
    x[0] = [-L, np.nextafter(2 * L, 0), -1e-300]
    x[-1, 1] = L
    want = np.where(x < 0, x + L, x)
    want = np.where(want >= L, want - L, want)
    want = np.where([bool(walls >> a & 1) for a in range(3)], x, want)
    p.set_state(x, 1.5)
    got, kappa = p.get_state()
    assert kappa == 1.5 and np.array_equal(got, want)
    for i, v in [(0, np.nan), (n - 1, 2 * L), (n // 2, -np.inf), (n - 1, np.nextafter(-L, -2 * L))]:
        bad = x.copy()
        bad[i, n % 3] = v
        with pytest.raises(rcp.RcpError):
            p.set_state(bad, 2.5)
        got, kappa = p.get_state()
        assert kappa == 1.5 and np.array_equal(got, want)
    m, v, o = p.get_optimizer()
    assert not m.any() and not v.any() and o["t"] == 0
    p.close()


def test_a_new_schedule_starts_every_packing_afresh(rcp, orc):
    # a batch of three whose schedules differ, run twice: the second run from
    # the same states gives the same bits, moments of the first run forgotten
    ds = [np.full(n, 0.5) + 0.01 * np.arange(n) / n for n in (40, 300, 2100)]
    Ls = [5.0, 8.0, 14.0]
    xs = [orc.rsa(d, L, 0.5, 3) for d, L in zip(ds, Ls)]
    sch = [rcp.schedule_from_rungs([(10.0 * (k + 1), 1e-3, 1e-3, 1.0, 1 << 30)]) for k in range(3)]

    def run(p, k0=0, some=slice(None)):
        for k, x in enumerate(xs[some]):
            p.set_state(x, 2.0, k)
        p.run_start(sch[some] if len(p.n) > 1 else sch[k0])
        p.run_continue(5)
        return [p.get_state(k) for k in range(len(p.n))]

    p = rcp.Packing(ds, Ls, 1.0, 0, init="none")
    a, b = run(p), run(p)
    p.close()
    for k in range(3):
        assert np.array_equal(a[k][0], b[k][0]) and a[k][1] == b[k][1]
        q = rcp.Packing(ds[k], Ls[k], 1.0, 0, init="none")
        c = run(q, k, slice(k, k + 1))
        q.close()
        assert np.array_equal(a[k][0], c[0][0]) and a[k][1] == c[0][1]


@pytest.mark.parametrize("graph_iters,step", [(1, 700), (4, 350), (8, 700), (32, 700), (32, 61)])
def test_iterations_do_not_depend_on_how_they_are_queued(rcp, orc, graph_iters, step):
    # several graphs in a row between two looks at the records, over list
    # builds, against one graph a look and single launches
    n, L = 300, 7.0
    d = 0.5 + 0.1 * np.arange(n) / n
    x = orc.rsa(d, L, 0.5, 5)

    def run(gi, st):
        p = rcp.Packing(d, L, 1.0, 0, init="none", tuning=rcp.make_tuning(graph_iters=gi))
        p.set_state(x, 1.2)
        p.run_start(rcp.schedule_from_rungs([(1e-4, 1e-3, 1e-4, 1.0, 1 << 30)]))
        for k in range(0, 700, st):
            p.run_continue(min(st, 700 - k))
        r = p.get_state() + p.get_optimizer()
        p.close()
        return r

    a, b = run(16, 16), run(graph_iters, step)
    # (the stop test holds before the last one)
    assert b[4]["iterations"] == a[4]["iterations"] > 600
    assert np.array_equal(a[0], b[0]) and a[1] == b[1]
    assert np.array_equal(a[2], b[2]) and np.array_equal(a[3], b[3])
