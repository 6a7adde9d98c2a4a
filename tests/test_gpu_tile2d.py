"""2-D steps in tiles against the oracle, where the tiling can go wrong: grids smaller than a
region or than four points, rows of every remainder, every order (whose groups of steps and rims
differ), more injected points or receivers in a region than it lists, more regions than CUs."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_side, has_gpu, oracle_side, rel_l2

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


def _check(shot, slots):
    import torch
    S, _ = oracle_side(shot)
    St, _ = oracle_side(shot, "true")
    fw = S.forward(want_traj=True)
    res = fw["data"] - St.forward()["data"]
    gref = S.gradient_full(fw["traj"], res)
    G, _ = gpu_side(shot)
    data, state = G.forward(want_state=True)
    assert np.any(fw["data"])
    assert rel_l2(data.cpu().numpy(), fw["data"]) <= 1e-5
    assert rel_l2(state[0].cpu().numpy(), fw["traj"][-1]) <= 1e-5
    rt = torch.as_tensor(res.astype(np.float32), device="cuda")
    full, _ = G.gradient(rt, G.slot_bytes * shot.nt)
    for m in slots:      # groups of other lengths, and levels read from slots
        g, _ = G.gradient(rt, G.slot_bytes * (m - 1))
        assert torch.equal(g, full), m
    assert rel_l2(full.cpu().numpy(), gref) <= 1e-4


def _shot(n, nbl, order, nt, seed=0):
    sh = W.random_layers(n, (10.0, 10.0), nbl, order, nt, np.random.default_rng(seed), 25.0)
    return W.replace(sh, vel_true=(sh.vel * 1.03).astype(np.float32))


@pytest.mark.parametrize("order", [2, 4, 6, 8, 10, 12, 14, 16])
@pytest.mark.parametrize("n,nbl", [((44, 25), 10), ((61, 90), 20), ((102, 43), 5), ((131, 33), 0)],
                         ids=["64", "101", "112", "131"])
def test_orders_and_row_remainders(n, nbl, order):
    _check(_shot(n, nbl, order, 67), (2, 7))


@pytest.mark.parametrize("n", [(3, 4), (2, 9), (5, 3), (4, 70)])
def test_grids_of_a_few_points(n):
    _check(_shot(n, 0, 2, 30), (3,))


@pytest.mark.parametrize("off", [0.0, 0.4])
def test_more_points_than_a_region_lists(off):
    """A receiver on (or beside) every point of a 40 x 40 patch."""
    sh = _shot((60, 56), 12, 8, 45)
    x, z = np.meshgrid(np.arange(8, 48), np.arange(4, 44))
    rec = np.stack([x.ravel(), z.ravel()], axis=1) * 10.0 + off * 10.0
    _check(W.replace(sh, rec=rec), (4,))


@pytest.mark.parametrize("order", [4, 8, 16])
def test_more_regions_than_compute_units(order):
    _check(_shot((1020, 790), 20, order, 13), (4,))


@pytest.mark.parametrize("order", [10, 16])
def test_wide_operators_on_large_grids_march(order):
    _check(_shot((1661, 1570), 20, order, 9), (3,))


@pytest.mark.parametrize("order", [12, 16])
def test_marched_steps_round_as_tiles(order):
    """A large grid's shot marches alone and runs in tiles in a batch: the same bits."""
    import torch
    from tests.test_gpu_batch import _batch, _device, _shots
    devs, dobs, _ = _device(_shots((1661, 1570), 90, order, 2, seed=order))
    dobs = [torch.zeros_like(d) for d in dobs]   # the models differ too deep to show in 90 steps
    budget = 10 * devs[0].slot_bytes
    phis, grads, dsims, _ = _batch(devs, dobs, budget, 0.0, 0.0)
    for i, d in enumerate(devs):
        phi, g, _, ds = d.misfit_gradient(dobs[i], budget, 0.0, want_dsim=True)
        assert phi > 0 and phis[i] == phi
        assert torch.equal(dsims[i], ds) and torch.equal(grads[i], g)
