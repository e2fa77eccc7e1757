"""fused_tail asked for together with the gradient kernels that have no such
form (variant bits 3 and 5): the iterations end and match the FP64 CPU oracle.

Bars: positions within 1e-9 of the step size per step plus 4e-16 L, kappa to
1e-12, as for the Adam steps elsewhere.
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


def _check_steps(rcp, orc, n, steps, phi=0.3, **tuning):
    rng = np.random.default_rng(n)
    d0 = 0.7 + 0.6 * rng.random(n)
    L = float((np.pi / 6 * np.sum(d0 ** 3) / phi) ** (1 / 3))
    x = rng.random((n, 3)) * L
    mu, ex, ek = 1e-4, 1e-3, 1e-4
    P = orc.default_params(d0, s=0.1, g=0.02)
    p = rcp.Packing(d0, L, 1.0, 0, init="none",
                    params=rcp.make_params(skin_s=0.1, skin_g=0.02, eps_x=P.eps_x),
                    tuning=rcp.make_tuning(**tuning))
    p.set_state(x, 1.0)
    p.adam_step(mu, ex, ek, steps)
    assert p.get_optimizer(moments=False)[2]["iterations"] == steps
    xg, kg = p.get_state()
    p.close()
    st = orc.RunState(x, d0, L, 1.0)
    orc.run(st, P, orc.oracle.absolute_schedule(mu, ex, ek, steps))
    d = np.abs(xg - st.x)
    d = np.minimum(d, L - d)
    assert d.max() <= 1e-9 * ex * steps + 4e-16 * L, d.max()
    assert kg == pytest.approx(st.kappa[0], rel=1e-12)


@pytest.mark.parametrize("graph", [1, 16])
@pytest.mark.parametrize("variant", [8, 9, 24, 32, 33, 32 + 128])
def test_fused_tail_with_kernels_that_have_none(rcp, orc, variant, graph):
    _check_steps(rcp, orc, 700, 10, fused_tail=1, variant=variant, graph_iters=graph)
