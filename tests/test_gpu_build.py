"""List builds at the sizes where the sort's digits and the search's splits
change: pair lists equal to the oracle's brute force, alone and in a batch."""
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


def _poly(n, seed):
    """n spheres in three size classes, and a box that holds them at 0.5."""
    rng = np.random.default_rng(seed)
    d = np.exp(rng.normal(0.0, 0.5, n))
    d[: max(1, n // 100)] *= 3.0
    L = max((np.pi / 6.0 * (d ** 3).sum() / 0.5) ** (1.0 / 3.0), 6.0 * d.max())
    return d, L, rng.uniform(0.0, L, (n, 3))


@pytest.mark.parametrize("n,skin", [
    (255, 0.3),      # one tile of keys, rows of 8 bits
    (256, 0.3), (257, 0.3), (512, 0.3),
    (513, 0.3),      # rows of 10 bits: three digits of 6 and 7
    (2048, 0.3), (2049, 0.3),     # one tile of keys, and one key more
    (6000, 0.3),     # rows of 13 bits: digits of 8 and 9
    (1500, 4.0),     # hundreds of pairs a sphere: staging fills many times
    (33000, 0.2),
])
def test_pairs_at_the_edges_of_digits_and_tiles(rcp, orc, n, skin):
    d, L, x = _poly(n, n)
    p = rcp.Packing(d, L, 1.0, 0, init="none", params=rcp.make_params(skin_s=skin, skin_g=0.02))
    p.set_state(x, 1.0)
    npairs = p.neighbor_build()
    gi, gj = p.pairs()
    p.close()
    oi, oj = orc.pairs_brute(x, d, L, 1.0, skin, 0.02)
    assert npairs == len(oi) > 0
    assert np.array_equal(gi, oi) and np.array_equal(gj, oj)


def test_pairs_of_a_batch(rcp, orc):
    # sizes of one to eighteen tiles share one sort and its digits
    ps = [_poly(n, 7 + n) for n in (40, 2048, 700, 36000, 2049, 9000)]
    p = rcp.Packing([d for d, _, _ in ps], [L for _, L, _ in ps], 1.0, 0, init="none",
                    params=rcp.make_params(skin_s=0.2, skin_g=0.02))
    for k, (_, _, x) in enumerate(ps):
        p.set_state(x, 1.0, k)
    p.run_start(rcp.schedule_from_rungs([(1e-5, 0.0, 0.0, 1.0, 1 << 30)]))
    p.run_continue(1)
    for k, (d, L, x) in enumerate(ps):
        gi, gj = p.pairs(k)
        oi, oj = orc.pairs_brute(x, d, L, 1.0, 0.2, 0.02)
        assert np.array_equal(gi, oi) and np.array_equal(gj, oj)
    p.close()


@pytest.mark.parametrize("n", [65536, 65537, 131073])   # 32 tiles of keys, one key more
def test_pairs_of_sampled_rows_at_the_longest_unscanned_sort(rcp, orc, n):
    d, L, x = _poly(n, 11)
    p = rcp.Packing(d, L, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.1, skin_g=0.02))
    p.set_state(x, 1.0)
    p.neighbor_build()
    gi, gj = p.pairs()
    p.close()
    rows = np.sort(np.random.default_rng(n).choice(n, 800, replace=False))
    want = orc.rows_pairs(x, d, L, 1.0, rows, 0.1, 0.02)
    i, j = np.concatenate([gi, gj]), np.concatenate([gj, gi])
    order = np.lexsort((j, i))
    i, j = i[order], j[order]
    for r, a, b, w in zip(rows, np.searchsorted(i, rows), np.searchsorted(i, rows, "right"), want):
        assert np.array_equal(j[a:b], w), int(r)


@pytest.mark.parametrize("n,skin", [(1, 0.3), (2, 0.3), (31, 0.3), (33, 4.0), (700, 3.0),
                                    (33000, 0.2)])
def test_shrink_scale_of_short_and_long_rows(rcp, orc, n, skin):
    # rows of none to hundreds of pairs, eight lanes a row
    d, L, x = _poly(n, 3 * n)
    if n <= 40:   # a cluster in a box that the listing cutoff fits
        L, x = 30.0 * d.max(), x / L * 3.0 * d.max()
    p = rcp.Packing(d, L, 1.0, 0, init="none", params=rcp.make_params(skin_s=skin, skin_g=0.02))
    p.set_state(x, 1.0)
    p.neighbor_build()
    kp, _ = p.shrink()
    p.close()
    i, j = orc.pairs_brute(x, d, L, 1.0, skin, 0.02)
    assert kp == orc.shrink(x, d, L, 1.0, i, j)
