"""Evaluations on several streams, and calls on the context's own stream after
them, with nothing waited for in between: each result is the one it has alone.
"""
import ctypes as C

import numpy as np
import pytest

import rcp_inputs as ri

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2608_12235_amd as m
    m.lib()
    return torch, m


def _outputs(torch, n):
    return [torch.zeros(s, dtype=torch.float64, device="cuda") for s in ((n, 3), (1,), (2,))]


def _queue(rcp, p, x, kappa, out, stream):
    """Gradient, then energy, queued on the stream."""
    h, st = p.handle, C.c_void_p(stream.cuda_stream)
    gx, gk, E = (C.c_void_p(o.data_ptr()) for o in out)
    xp = C.c_void_p(x.data_ptr())
    rcp.api.check(rcp.lib().rcp_adjoint_dev(h, xp, kappa, 0.1, gx, gk, st))
    rcp.api.check(rcp.lib().rcp_energy_dev(h, xp, kappa, 0.1, E, st))


@pytest.mark.parametrize("n,wide", [(3000, False), (200003, False), (200003, True)])
def test_evaluations_on_several_streams(env, n, wide):
    torch, rcp = env
    w = ri.small_polydisperse(n, 4.0, 0.3, seed=3)
    p = rcp.Packing(w.d0, w.L, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.5),
                    tuning=rcp.make_tuning(variant=224, item_work=3072) if wide else None)
    p.set_state(w.x, 1.0)
    p.neighbor_build()
    rng = np.random.default_rng(5)
    # five sets of positions at which the list holds
    xs = [torch.tensor(np.mod(w.x + rng.uniform(-0.05, 0.05, w.x.shape) * w.d0.min(), w.L),
                       device="cuda") for _ in range(5)]
    streams = [torch.cuda.Stream() for _ in xs]
    alone, builds = [], p.stats()["rebuilds"]
    for x, s in zip(xs, streams):
        out = _outputs(torch, n)
        torch.cuda.synchronize()
        _queue(rcp, p, x, 1.0, out, s)
        torch.cuda.synchronize()
        alone.append(out)
    home = p.energy_grad(mu=0.1)
    outs = [_outputs(torch, n) for _ in xs]
    torch.cuda.synchronize()
    for _ in range(4):
        for x, o, s in zip(xs, outs, streams):
            _queue(rcp, p, x, 1.0, o, s)
        # on the context's own stream, at its own positions
        e = p.energy_grad(mu=0.1)
        assert e["E_overlap"] == home["E_overlap"] and np.array_equal(e["g"], home["g"])
    torch.cuda.synchronize()
    for a, o in zip(alone, outs):
        for u, v in zip(a, o):
            assert torch.equal(u, v)
    assert p.stats()["rebuilds"] == builds
    p.close()


def test_a_new_state_does_not_reach_an_evaluation_in_flight(env):
    # positions handed in and steps taken right after an evaluation was queued
    # at the packing's own positions (its list was built for them)
    torch, rcp = env
    n = 200003
    w = ri.small_polydisperse(n, 4.0, 0.3, seed=4)
    x2 = np.mod(w.x + 0.3, w.L)
    x = torch.tensor(w.x, device="cuda")
    want = None
    for rep in range(4):
        p = rcp.Packing(w.d0, w.L, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.5))
        out, s = _outputs(torch, n), torch.cuda.Stream()
        torch.cuda.synchronize()
        st = C.c_void_p(s.cuda_stream)
        gx, gk, _ = (C.c_void_p(o.data_ptr()) for o in out)
        rcp.api.check(rcp.lib().rcp_adjoint_dev(p.handle, C.c_void_p(x.data_ptr()), 1.0, 0.1, gx, gk,
                                                st))
        if rep == 0:
            torch.cuda.synchronize()
        elif rep == 1:
            p.set_state(x2, 1.0)
        elif rep == 2:
            p.adam_step(1e-4, 1e-2, 1e-4, 20)
        else:
            p.set_tuning(rcp.make_tuning(row_cost=9, item_work=600))
        torch.cuda.synchronize()
        if want is None:
            want = [o.clone() for o in out]
        assert torch.equal(want[0], out[0]) and torch.equal(want[1], out[1]), rep
        p.close()
