"""Energy, gradient and steps under work items of more rows than a wave has lanes
(variant bit 5, item_work above 256 row_cost), against the FP64 CPU oracle.

Sparse packings, whose items hold up to 128 rows.  Bars: 1e-10 per component of
the summed |contributions| and 1e-10 of the sums; positions after Adam steps
within 1e-9 of the step size per step plus 4e-16 L, kappa to 1e-12, as
elsewhere.
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


def _packing(rcp, n, row_cost, item_work, variant, orc=None, phi=0.12):
    rng = np.random.default_rng(n)
    d0 = 0.7 + 0.6 * rng.random(n)
    L = float((np.pi / 6 * np.sum(d0 ** 3) / phi) ** (1 / 3))
    eps = {"eps_x": orc.default_params(d0, s=0.05, g=0.02).eps_x} if orc else {}
    p = rcp.Packing(d0, L, 1.0, 0, init="none",
                    params=rcp.make_params(skin_s=0.05, skin_g=0.02, **eps),
                    tuning=rcp.make_tuning(row_cost=row_cost, item_work=item_work, variant=variant))
    return p, d0, L, rng.random((n, 3)) * L


def _check(orc, x, d0, L, kappa, mu, e):
    pi, pj = orc.pairs_brute(x, d0, L, kappa, 0.0, 0.0)
    r = orc.energy_grad(x, d0, L, kappa, mu, pi, pj)
    assert e["n_overlap"] == r["n_overlap"] > len(d0) // 10
    assert e["E_overlap"] == pytest.approx(r["E_ov"], rel=1e-10)
    assert e["dE_dkappa_overlap"] == pytest.approx(r["gk_ov"], rel=1e-10)
    assert np.all(np.abs(e["g"] - r["g"]) <= 1e-10 * r["gscale"])
    return r


@pytest.mark.parametrize("n", [6500, 20011])
@pytest.mark.parametrize("row_cost,item_work,variant", [(6, 3072, 224), (1, 512, 33), (4, 2048, 32)])
def test_energy_under_wide_items(rcp, orc, n, row_cost, item_work, variant):
    p, d0, L, x = _packing(rcp, n, row_cost, item_work, variant)
    p.set_state(x, 1.0)
    _check(orc, x, d0, L, 1.0, 0.3, p.energy_grad(mu=0.3))
    # a run that ends on its limit evaluates the state it leaves
    r = p.inflate_run(rcp.schedule_from_rungs([(1e-4, 1e-3, 1e-4, 1.0, 100)]), max_iters=3)[0]
    xg, kg = p.get_state()
    p.close()
    pi, pj = orc.pairs_brute(xg, d0, L, kg, 0.0, 0.0)
    o = orc.energy_grad(xg, d0, L, kg, 0.0, pi, pj)
    assert r["energy"] == pytest.approx(o["E_ov"], rel=1e-10)
    assert r["max_overlap"] == pytest.approx(o["max_delta"], rel=1e-10)


def test_differentiable_energy_under_wide_items(rcp, orc):
    import torch
    p, d0, L, x = _packing(rcp, 8000, 6, 3072, 224)
    p.set_state(x, 1.0)
    p.neighbor_build()
    xt = torch.tensor(x, device="cuda", requires_grad=True)
    kap = torch.tensor(1.0, dtype=torch.float64, requires_grad=True)
    E, worst = rcp.overlap_energy(xt, kap, p, mu=0.3)
    E.backward()
    pi, pj = orc.pairs_brute(x, d0, L, 1.0, 0.0, 0.0)
    r = orc.energy_grad(x, d0, L, 1.0, 0.3, pi, pj)
    assert float(E.detach()) == pytest.approx(r["E_ov"] + r["E_growth"], rel=1e-10)
    assert float(worst.detach()) == pytest.approx(r["max_delta"], rel=1e-10)
    assert np.all(np.abs(xt.grad.cpu().numpy() - r["g"]) <= 1e-10 * r["gscale"])
    p.close()


@pytest.mark.parametrize("variant", [32, 40, 41, 62])
def test_steps_of_wide_items(rcp, orc, variant):
    # bits 1 to 4 do not apply with bit 5: the kernel of 512 rows an item runs
    p, d0, L, x = _packing(rcp, 9001, 6, 3072, variant, orc)
    mu, ex, ek, steps = 1e-4, 1e-3, 1e-4, 5
    p.set_state(x, 1.0)
    p.adam_step(mu, ex, ek, steps)
    xg, kg = p.get_state()
    p.close()
    st = orc.RunState(x, d0, L, 1.0)
    orc.run(st, orc.default_params(d0, s=0.05, g=0.02), orc.oracle.absolute_schedule(mu, ex, ek, steps))
    d = np.abs(xg - st.x)
    d = np.minimum(d, L - d)
    assert d.max() <= 1e-9 * ex * steps + 4e-16 * L, d.max()
    assert kg == pytest.approx(st.kappa[0], rel=1e-12)


def test_a_new_cut_of_a_built_list_has_items_for_every_row(rcp, orc):
    # 2000 spheres: the table is laid out for 16000 entries, and with the
    # default cut it holds this list of a few more; a cut of one unit an item
    # needs an item for each of them
    rng = np.random.default_rng(7)
    d0 = 0.7 + 0.6 * rng.random(2000)
    L = float((np.pi / 6 * np.sum(d0 ** 3) / 0.4) ** (1 / 3))
    x = rng.random((2000, 3)) * L
    p = rcp.Packing(d0, L, 1.0, 0, init="none", params=rcp.make_params(skin_s=0.28, skin_g=0.02))
    p.set_state(x, 1.0)
    assert 16000 + 500 < 2 * p.neighbor_build() < 16000 + 1300
    p.set_tuning(rcp.make_tuning(row_cost=1, item_work=1))
    _check(orc, x, d0, L, 1.0, 0.3, p.energy_grad(mu=0.3))
    assert p.stats()["rebuilds"] == 1
    p.close()
