"""rcp_energy_dev_static against rcp_energy_dev, whose bits it gives, over the
kinds of packing and of work items; the packing's state is left as it was.
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


@pytest.mark.parametrize("kind,n", [
    ("plain", 2), ("plain", 300), ("plain", 5000), ("plain", 60001), ("plain", 200003),
    ("plain", 1000003), ("frozen", 5000), ("walls", 5000), ("wide", 300), ("wide", 60001),
    ("wider", 400003), ("thin", 60001), ("parked", 60001)])
def test_the_same_bits_without_allocation(env, kind, n):
    torch, rcp = env
    lib = rcp.lib()
    if n == 2:
        w = ri.small_polydisperse(2, 1.5, 0.002, seed=1)
        w.x[:] = [[0.5, 0.5, 0.5], [0.5 + 0.8 * w.d0.mean(), 0.5, 0.5]]
    else:
        w = ri.small_polydisperse(n, 20.0 if n > 1000 else 2.0, 0.5, seed=n, family="powerlaw")
    # (thin and wider: more blocks than a portion of the fixed array holds)
    tuning = {"wide": dict(variant=224, item_work=3072),
              "wider": dict(variant=224, row_cost=1, item_work=512),
              "thin": dict(row_cost=1, item_work=1)}.get(kind)
    parked = kind == "parked"
    p = rcp.Packing([w.d0, np.ones(30)] if parked else w.d0, [w.L, w.L] if parked else w.L, 1.0, 0,
                    init="none", params=rcp.make_params(skin_s=0.5),
                    boundary=(5, 0) if kind == "walls" else None,
                    tuning=rcp.make_tuning(**tuning) if tuning else None)
    p.set_state(w.x, 1.0)
    if kind == "frozen":
        p.set_frozen(np.arange(n) % 3 == 0)
    if parked:
        p.set_state(np.random.default_rng(1).random((30, 3)) * w.L, 1.0, 1)
        p.inflate_run([rcp.schedule_from_rungs([(1e-4, 1e-6, 0.0, 1.0, b)]) for b in (3, 200)])
    else:
        p.neighbor_build()
    x, kappa = p.get_state()
    rng = np.random.default_rng(n)
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    for step in (0.0, 0.05, 0.1):
        xt = x + step * w.d0.min() * rng.uniform(-1, 1, x.shape)
        if kind != "walls":
            xt = np.mod(xt, w.L)
        xt = torch.tensor(xt, device="cuda")
        e = torch.zeros((2, 2), dtype=torch.float64, device="cuda")
        args = (p.handle, C.c_void_p(xt.data_ptr()), kappa, 0.0)
        # (first without what an allocating call may leave behind)
        rcp.api.check(lib.rcp_energy_dev_static(*args, C.c_void_p(e[0].data_ptr()), stream))
        rcp.api.check(lib.rcp_energy_dev(*args, C.c_void_p(e[1].data_ptr()), stream))
        a, b = e.cpu().numpy()
        assert a[0] > 0.0 and np.array_equal(a, b), (step, a, b)
    xa, ka = p.get_state()
    assert np.array_equal(xa, x) and ka == kappa
    p.close()


def test_steps_after_a_static_energy(env):
    # the call leaves no trace in the steps that follow it, whichever of the
    # two position buffers is the current one
    torch, rcp = env
    w = ri.small_polydisperse(5000, 20.0, 0.5, seed=2, family="powerlaw")

    def steps(static, variant):
        p = rcp.Packing(w.d0, w.L, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.5),
                        tuning=rcp.make_tuning(variant=variant))
        p.set_state(w.x, 1.0)
        p.set_frozen(np.arange(5000) % 3 == 0)
        e = torch.zeros(2, dtype=torch.float64, device="cuda")
        for k in range(4):
            p.adam_step(1e-4, 1e-5, 1e-6, 1 + k % 2)
            if static:
                x, kappa = p.get_state()
                xt = torch.tensor(np.mod(x + 0.1 * w.d0.min(), w.L), device="cuda")
                rcp.api.check(rcp.lib().rcp_energy_dev_static(
                    p.handle, C.c_void_p(xt.data_ptr()), kappa, 0.0, C.c_void_p(e.data_ptr()),
                    C.c_void_p(torch.cuda.current_stream().cuda_stream)))
        out = p.get_state(diameters=True)
        p.close()
        return out

    for variant in (192, 64):
        a, b = steps(False, variant), steps(True, variant)
        assert np.array_equal(a[0], b[0]) and a[1] == b[1] and np.array_equal(a[2], b[2])
