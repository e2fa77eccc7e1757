"""Calls that run out of room leave the context as it was: a work table that
would be too large, a list that would be too long.
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


def _poly(n, phi, seed):
    rng = np.random.default_rng(seed)
    d = 0.7 + 0.6 * rng.random(n)
    L = float((np.pi / 6 * np.sum(d ** 3) / phi) ** (1 / 3))
    return d, L, rng.random((n, 3)) * L


def test_a_cut_with_too_many_items_is_refused(rcp):
    # 65536 units a row and one an item: 1000 spheres take 1.1e7 blocks, 1e5
    # more than a table has
    ps = [_poly(n, 0.3, n) for n in (1000, 100000)]

    def run(refused):
        p = rcp.Packing([d for d, _, _ in ps], [L for _, L, _ in ps], 1.0, 0, init="none",
                        params=rcp.make_params(skin_s=0.3))
        for k, (_, _, x) in enumerate(ps):
            p.set_state(x, 1.0, k)
            p.neighbor_build(k)
        if refused:
            with pytest.raises(rcp.RcpError, match="work table"):
                p.set_tuning(rcp.make_tuning(row_cost=65536, item_work=1))
        e = [p.energy_grad(mu=0.1, k=k) for k in range(2)]
        p.adam_step(1e-4, 1e-3, 1e-4, 3)
        out = e + [p.get_state(k) for k in range(2)]
        p.close()
        return out

    a, b = run(False), run(True)
    for k in range(2):
        assert np.array_equal(a[k]["g"], b[k]["g"]) and a[k]["E_overlap"] == b[k]["E_overlap"]
        assert np.array_equal(a[2 + k][0], b[2 + k][0]) and a[2 + k][1] == b[2 + k][1]
