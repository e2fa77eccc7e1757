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


def test_a_list_too_long_is_refused(rcp, orc):
    # 7e4 spheres within a reach of almost half the box: 2.4e9 entries, more
    # than 32-bit row pointers address.  The build stops after its sort;
    # positions, diameters and moments are still the spheres' own, and with a
    # smaller skin the list is the right one.
    rng = np.random.default_rng(3)
    n, L = 70000, 100.0
    d = 0.9 + 0.2 * rng.random(n)
    x = rng.random((n, 3)) * L
    p = rcp.Packing(d, L, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.3, skin_g=0.02))
    p.set_state(x, 1.0)
    frozen = np.zeros(n, np.uint8)
    frozen[::2] = 1
    p.set_frozen(frozen)
    p.adam_step(1e-4, 1e-3, 1e-4, 3)
    before = p.get_state(diameters=True)
    m, v, o = p.get_optimizer()
    p.set_skin(26.6, 0.02)
    for _ in range(2):
        with pytest.raises(rcp.RcpError, match="neighbour list"):
            p.neighbor_build()
        after = p.get_state(diameters=True)
        assert np.array_equal(after[0], before[0]) and after[1] == before[1]
        assert np.array_equal(after[2], before[2])
        m2, v2, o2 = p.get_optimizer()
        assert np.array_equal(m, m2) and np.array_equal(v, v2) and o == o2
    p.set_skin(0.3, 0.02)
    e = p.energy_grad(mu=0.3)
    kappa = before[1]
    try:
        orc.set_frozen(frozen)
        pi, pj = orc.pairs_cells(before[0], d, L, 1.01, 0.0, 0.02)
        r = orc.energy_grad(before[0], d, L, kappa, 0.3, pi, pj)
    finally:
        orc.set_frozen(None)
    assert e["n_overlap"] == r["n_overlap"] > 1000
    assert e["E_overlap"] == pytest.approx(r["E_ov"], rel=1e-10)
    assert np.all(np.abs(e["g"] - r["g"]) <= 1e-10 * r["gscale"])
    p.close()
