"""Seating where the seating distance leaves one, two or three grid cells per
axis: bit for bit the FP64 CPU oracle's, which tests every frozen sphere.
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
@pytest.mark.parametrize("seed", [1, 2, 3])
@pytest.mark.parametrize("nc,k0", [(1, 0.58), (2, 0.4), (2, 0.26), (3, 0.21), (4, 0.05)])
def test_seating_with_few_cells_per_axis(rcp, orc, nc, k0, seed, dim):
    # two frozen spheres of 0.44 L, the others seated at diameters k0 L and less
    L, nf, n = 10.0, 2, 300
    rng = np.random.default_rng(seed)
    d0 = np.concatenate([np.full(nf, 4.4), 4.0 * (0.5 + 0.5 * rng.random(n))])
    d0[nf] = 4.0
    kappa = k0 * L / 4.0
    assert int(L / (0.5 * (4.4 + kappa * 4.0))) == nc
    x = np.zeros((nf + n, dim))
    x[:nf] = rng.random((nf, dim)) * L
    mask = np.zeros(nf + n, np.uint8)
    mask[:nf] = 1
    p = rcp.Packing(d0, L, 1.0, 0, init="none", dim=dim,
                    params=rcp.make_params(skin_s=0.01, skin_g=0.0))
    p.set_state(x, 1.0)
    p.set_frozen(mask)
    p.seat(kappa, 10 + seed)
    xg, kg = p.get_state()
    p.close()
    assert kg == kappa
    x3 = np.zeros((nf + n, 3))
    x3[:, :dim] = x
    try:
        if dim == 2:
            orc.set_dim(2)
        orc.set_frozen(mask)
        xo = orc.seat(x3, d0, L, kappa, 10 + seed)
    finally:
        orc.set_frozen(None)
        if dim == 2:
            orc.set_dim(3)
    assert np.array_equal(xg, xo[:, :dim])
