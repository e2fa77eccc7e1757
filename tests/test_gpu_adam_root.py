"""The root of a second moment below 1e-200 in the Adam step is the correctly
rounded one.

A sphere at x = 0 without contacts and with beta1 = beta2 = 1/2 takes, at t = 1,
exactly the step eta m / (sqrt(v) + eps_x): the bias corrections cancel the
decay.  With v = s^2 (s of 26 bits, so the square is exact) and eps_x far below
s the denominator is s if the root is right; with v = 0 and eps_x = s it is s
without one.  The two steps must have the same bits.
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


def _step(rcp, eps, m, v):
    n, L = 4, 20.0
    p = rcp.Packing(np.ones(n), L, 1.0, 0, init="none",
                    params=rcp.make_params(beta1=0.5, beta2=0.5, eps_x=eps))
    x = np.zeros((n, 3))
    x[:, 1] = 5.0 * np.arange(n)
    p.set_state(x, 1.0)
    o = p.get_optimizer(moments=False)[2]
    m3, v3 = np.zeros((n, 3)), np.zeros((n, 3))
    m3[:, 0], v3[:, 0] = m, v
    p.set_optimizer(o, m3, v3)
    p.adam_step(0.0, 2.0 ** -6, 0.0, 1)
    xg = p.get_state()[0]
    p.close()
    assert np.array_equal(xg[:, 1:], x[:, 1:])
    return xg[:, 0]


@pytest.mark.parametrize("exponent", [-360, -365, -420, -500])
def test_root_of_tiny_second_moments(rcp, exponent):
    rng = np.random.default_rng(-exponent)
    for _ in range(24):
        s = float(rng.integers(1 << 25, 1 << 26)) * 2.0 ** exponent
        assert 0.0 < s * s < 1e-200
        m = -s * rng.uniform(0.5, 1.5, 4)
        a, b = _step(rcp, s, m, 0.0), _step(rcp, s * 2.0 ** -80, m, s * s)
        assert np.all(a > 0.0) and np.allclose(a, -m / s * 2.0 ** -6, rtol=1e-12)
        assert np.array_equal(a, b), (s, a, b)
