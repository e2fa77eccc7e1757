"""A census in which one packing has frozen spheres, one has walls and one has
neither: each takes the steps it would take in a context of its own, against
the FP64 CPU oracle.

Bars: positions within 1e-9 of the step size per step plus 4e-16 L, kappa to
1e-12, as for the Adam steps elsewhere; frozen spheres stay where they are.
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


@pytest.mark.parametrize("dim", [3, 2])
@pytest.mark.parametrize("graph", [1, 8])
def test_frozen_and_walled_packings_in_one_census(rcp, orc, dim, graph):
    rng = np.random.default_rng(40 + dim)
    ns = [900, 700, 400]
    d0s = [0.7 + 0.6 * rng.random(n) for n in ns]
    unit = np.pi / 6 if dim == 3 else np.pi / 4
    Ls = [float((unit * np.sum(d ** dim) / 0.4) ** (1 / dim)) for d in d0s]
    xs = [0.7 + rng.random((n, dim)) * (L - 1.4) for n, L in zip(ns, Ls)]
    frozen = np.zeros(ns[0], np.uint8)
    frozen[::3] = 1
    bnds = [(0, 0), (1, 0), (0, 0)]
    mu, ex, ek, steps = 1e-4, 1e-3, 1e-4, 6
    eps = orc.default_params(d0s[0], s=0.3, g=0.02).eps_x
    p = rcp.Packing(d0s, Ls, 1.0, 0, init="none", dim=dim, boundary=bnds,
                    params=rcp.make_params(skin_s=0.3, skin_g=0.02, eps_x=eps),
                    tuning=rcp.make_tuning(graph_iters=graph))
    for k, x in enumerate(xs):
        p.set_state(x, 1.0, k)
    p.set_frozen(frozen)
    p.adam_step(mu, ex, ek, steps)
    got = [p.get_state(k) for k in range(3)]
    p.close()
    assert np.array_equal(got[0][0][frozen == 1], xs[0][frozen == 1])
    for k in range(3):
        x3 = np.zeros((ns[k], 3))
        x3[:, :dim] = xs[k]
        P = orc.default_params(d0s[k], s=0.3, g=0.02)
        P.eps_x = eps
        try:
            if dim == 2:
                orc.set_dim(2)
            if k == 0:
                orc.set_frozen(frozen)
            orc.set_boundary(*bnds[k])
            st = orc.RunState(x3, d0s[k], Ls[k], 1.0)
            orc.run(st, P, orc.oracle.absolute_schedule(mu, ex, ek, steps))
        finally:
            orc.set_frozen(None)
            orc.set_boundary(0, 0)
            if dim == 2:
                orc.set_dim(3)
        d = np.abs(got[k][0] - st.x[:, :dim])
        if bnds[k] == (0, 0):
            d = np.minimum(d, Ls[k] - d)
        assert d.max() <= 1e-9 * ex * steps + 4e-16 * Ls[k], (k, d.max())
        assert got[k][1] == pytest.approx(st.kappa[0], rel=1e-12)
