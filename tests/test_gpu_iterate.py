"""The wave-per-item gradient + Adam kernel at the edges of its work items,
against the FP64 CPU oracle.

A large sphere with `k` small partners gives one row of k entries beside k
rows of a few: k below, at and above a round of 64 entries, two rounds, the
512 entries from which a block shares its items, and many times that.  The
cuts run from one row an item to 64 and to items of thousands of entries.
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


def _star(k, dim, seed):
    """One sphere of diameter 8 at the centre, k of diameter 0.8 to 1.2 whose
    centres lie on a shell they overlap it from, 37 more in a corner."""
    rng = np.random.default_rng(seed)
    L, big = 24.0, 8.0
    u = rng.standard_normal((k, dim))
    u /= np.linalg.norm(u, axis=1)[:, None]
    d = 0.8 + 0.4 * rng.random(k + 37)
    x = np.concatenate([np.full((1, dim), 0.5 * L),
                        0.5 * L + u * (0.45 * big + 0.4 * d[:k, None]),
                        rng.random((37, dim)) * 4.0])
    return np.concatenate([[big], d]), x, L


@pytest.mark.parametrize("k", [1, 62, 63, 64, 65, 128, 129, 511, 512, 513, 4000])
@pytest.mark.parametrize("row_cost,item_work,kind", [
    (6, 1536, "plain"), (6, 1536, "frozen"), (6, 1536, "walls"), (6, 1536, "disks"),
    (1, 1, "plain"), (4, 1024, "plain"), (64, 16384, "plain"), (6, 3072, "wide")])
def test_long_rows_and_item_cuts(rcp, orc, k, row_cost, item_work, kind):
    if kind != "plain" and k not in (64, 513, 4000):
        pytest.skip("plain packings run every length")
    dim = 2 if kind == "disks" else 3
    d0, x, L = _star(k, dim, 17 + k)
    mu, ex, ek, steps = 1e-4, 1e-3, 1e-4, 3
    frozen = np.zeros(len(d0), np.uint8)
    if kind in ("frozen", "wide"):
        frozen[0] = 1
        frozen[2::5] = 1
    bnd = (7, 0) if kind == "walls" else None
    P = orc.default_params(d0, s=0.3, g=0.02)
    p = rcp.Packing(d0, L, 1.0, 0, init="none", dim=dim, boundary=bnd,
                    params=rcp.make_params(skin_s=0.3, skin_g=0.02, eps_x=P.eps_x),
                    tuning=rcp.make_tuning(row_cost=row_cost, item_work=item_work,
                                           variant=192 | (32 if kind == "wide" else 0)))
    p.set_state(x, 1.0)
    if frozen.any():
        p.set_frozen(frozen)
    p.adam_step(mu, ex, ek, steps)
    xg, kg = p.get_state()
    assert p.stats()["max_degree"] >= k
    p.close()
    x3 = np.zeros((len(d0), 3))
    x3[:, :dim] = x
    try:
        if dim == 2:
            orc.set_dim(2)
        if frozen.any():
            orc.set_frozen(frozen)
        if bnd:
            orc.set_boundary(*bnd)
        st = orc.RunState(x3, d0, L, 1.0)
        orc.run(st, P, orc.oracle.absolute_schedule(mu, ex, ek, steps))
    finally:
        orc.set_frozen(None)
        orc.set_boundary(0, 0)
        if dim == 2:
            orc.set_dim(3)
    d = np.abs(xg - st.x[:, :dim])
    if bnd is None:
        d = np.minimum(d, L - d)
    assert d.max() <= 1e-9 * ex * steps + 4e-16 * L, d.max()
    assert kg == pytest.approx(st.kappa[0], rel=1e-12)


@pytest.mark.parametrize("k", [1, 64, 513, 4000])
@pytest.mark.parametrize("kind", ["plain", "frozen", "walls", "parked"])
def test_energy_of_long_rows(rcp, orc, k, kind):
    # the evaluation by work items: 1e-10 per component of the summed
    # |contributions|, as elsewhere.  "parked": the packing of a census that
    # finished first has given up its items, and its rows are cut again.
    d0, x, L = _star(k, 3, 29 + k)
    frozen = np.zeros(len(d0), np.uint8)
    bnd = (7, 0) if kind == "walls" else None
    if kind == "parked":
        p = rcp.Packing([d0, np.ones(30)], [L, L], 1.0, 0, init="none")
        p.set_state(x, 1.0, 0)
        p.set_state(np.random.default_rng(1).random((30, 3)) * L, 1.0, 1)
        p.inflate_run([rcp.schedule_from_rungs([(1e-4, 1e-4, 0.0, 1.0, b)]) for b in (3, 200)])
        x, kappa = p.get_state(0)
    else:
        p = rcp.Packing(d0, L, 1.0, 0, init="none", boundary=bnd)
        p.set_state(x, 1.0)
        kappa = 1.0
        if kind == "frozen":
            frozen[0] = 1
            frozen[2::5] = 1
            p.set_frozen(frozen)
    e = p.energy_grad(mu=0.3)
    p.close()
    try:
        if kind == "frozen":
            orc.set_frozen(frozen)
        if bnd:
            orc.set_boundary(*bnd)
        pi, pj = orc.pairs_brute(x, d0, L, kappa, 0.0, 0.0)
        r = orc.energy_grad(x, d0, L, kappa, 0.3, pi, pj)
    finally:
        orc.set_frozen(None)
        orc.set_boundary(0, 0)
    assert e["n_overlap"] == r["n_overlap"] and r["n_overlap"] >= k
    assert e["E_overlap"] == pytest.approx(r["E_ov"], rel=1e-10)
    assert e["dE_dkappa_overlap"] == pytest.approx(r["gk_ov"], rel=1e-10)
    assert np.all(np.abs(e["g"] - r["g"]) <= 1e-10 * r["gscale"])


@pytest.mark.parametrize("n", [3, 300, 3000, 70000])
def test_tail_placement_changes_nothing(rcp, n):
    # the tail at the start of the next kernel (one packing of up to 1024
    # blocks), as a launch of its own (launches timed, one iteration a
    # launch), and beside packings of another size that end early and late:
    # the same bits
    def packing(ns, **kw):
        ds = [0.7 + 0.6 * np.random.default_rng(m).random(m) for m in ns]
        Ls = [float((np.pi / 6 * np.sum(d ** 3) / 0.55) ** (1 / 3)) if m > 3 else 9.0
              for m, d in zip(ns, ds)]
        p = rcp.Packing(ds, Ls, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.4),
                        tuning=rcp.make_tuning(**kw))
        for k, (m, L) in enumerate(zip(ns, Ls)):
            p.set_state(np.random.default_rng(100 + m).random((m, 3)) * L, 1.0, k)
        # rung ends, a cap and a list build fall inside the graphs
        p.inflate_run([rcp.schedule_from_rungs([(1e-3, 3e-3, 3e-4, 1.0, 9 + m % 5),
                                                (1e-4, 2e-3, 2e-4, 0.99, 12)]) for m in ns])
        out = [p.get_state(k) for k in range(len(ns))] + [p.get_optimizer(k) for k in range(len(ns))]
        p.close()
        return out
    a = packing([n])
    for kw in (dict(graph_iters=1), dict(graph_iters=7), dict(time_kernels=2)):
        b = packing([n], **kw)
        assert np.array_equal(a[0][0], b[0][0]) and a[0][1] == b[0][1], kw
        assert np.array_equal(a[1][0], b[1][0]) and np.array_equal(a[1][1], b[1][1])
        assert a[1][2] == b[1][2]
    m = 400 if n < 1000 else 900
    for kw in (dict(graph_iters=8), dict(graph_iters=8, time_kernels=1)):
        b = packing([m, n, m + 1], **kw)
        assert np.array_equal(a[0][0], b[1][0]) and a[0][1] == b[1][1], kw
        assert np.array_equal(a[1][0], b[4][0]) and a[1][2] == b[4][2]
