"""2-D steps that march (large grids, by order and kind of call) against the tiles, bit for bit,
and the adjoint of the source against the oracle on both sides of its rule."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_side, has_gpu, oracle_side, rel_l2

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


def _near_source(sh, half, step, off):
    """Receivers in a patch around the source, where a few steps show."""
    cx, cz = sh.src[0]
    ax = np.arange(-half, half + 1) * step * 10.0 + off
    x, z = np.meshgrid(cx + ax, np.maximum(cz + ax, 0.0))
    return W.replace(sh, rec=np.stack([x.ravel(), z.ravel()], axis=1))


def _pair(n, nt, order, half, step, off):
    from tests.test_gpu_batch import _device, _shots
    shots = [_near_source(sh, half, step, off) for sh in _shots(n, nt, order, 2, seed=order)]
    return _device(shots)


@pytest.mark.parametrize("n,order", [((3650, 3600), 6), ((2850, 2900), 8), ((980, 970), 10), ((1000, 961), 16)])
def test_marched_forward_has_the_tiles_bits(n, order):
    """A forward call marches; the same shot's data in a batch comes from tiles."""
    import torch
    from tests.test_gpu_batch import _batch
    devs, dobs, _ = _pair(n, 9, order, 4, 2, 3.0)
    zero = [torch.zeros_like(d) for d in dobs]
    _, _, dsims, _ = _batch(devs, zero, 10 * devs[0].slot_bytes, 0.0, 0.0)
    for d, ds in zip(devs, dsims):
        data = d.forward()
        assert torch.count_nonzero(data) > 100 and torch.equal(data, ds)


@pytest.mark.parametrize("half,off", [(6, 0.0), (6, 4.0), (40, 4.0)], ids=["nodes", "between", "many"])
def test_marched_gradient_injects_as_tiles(half, off):
    """Residuals injected by the marching workgroups and, at more points than those look
    through (6,561), by a launch of their own."""
    import torch
    from tests.test_gpu_batch import _batch
    devs, dobs, _ = _pair((1220, 1200), 12, 16, half, 1, off)
    zero = [torch.zeros_like(d) for d in dobs]
    budget = 4 * devs[0].slot_bytes
    phis, grads, dsims, _ = _batch(devs, zero, budget, 0.0, 0.0)
    for i, d in enumerate(devs):
        phi, g, _, ds = d.misfit_gradient(zero[i], budget, 0.0, want_dsim=True)
        assert phi > 0 and phis[i] == phi
        assert torch.equal(dsims[i], ds) and torch.equal(grads[i], g)


def test_batch_of_one_runs_in_tiles():
    """On a grid whose solo calls march, in place: the same bits."""
    import torch
    from tests.test_gpu_batch import _batch
    devs, dobs, _ = _pair((1220, 1200), 12, 16, 6, 1, 4.0)
    zero = torch.zeros_like(dobs[0])
    budget = 4 * devs[0].slot_bytes
    phi, g, _, ds = devs[0].misfit_gradient(zero, budget, 0.0, want_dsim=True)
    phis, grads, dsims, _ = _batch(devs[:1], [zero], budget, 0.0, 0.0)
    assert phis[0] == phi and torch.equal(dsims[0], ds) and torch.equal(grads[0], g)


@pytest.mark.parametrize("n,order", [((60, 50), 4), ((960, 870), 4), ((760, 770), 16), ((350, 360), 16), ((901, 870), 8)])
def test_adjoint_of_the_source(n, order):
    import torch
    sh = W.random_layers(n, (10.0, 10.0), 20, order, 24, np.random.default_rng(order), 25.0)
    sh = _near_source(sh, 5, 2, 4.0)
    S, _ = oracle_side(sh)
    G, _ = gpu_side(sh)
    r = np.random.default_rng(1).standard_normal((sh.nt + 1, len(sh.rec))).astype(np.float32)
    ref = S.adjoint_src(r.astype(np.float64))
    assert np.any(ref)
    assert rel_l2(G.adjoint_src(torch.as_tensor(r, device="cuda")).cpu().numpy(), ref) <= 1e-4


@pytest.mark.parametrize("nbl", [1, 2])
def test_thin_layers_divide_alike(nbl):
    """Marched steps divide by 1 + a, tiles multiply by its corrected reciprocal.  At the stability
    limit a layer of one cell has 1 + a up to 6.6 at order 10; source and receivers lie at its corner."""
    import torch
    from tests.test_gpu_batch import _batch, _device, _shots
    shots = []
    for sh in _shots((1018, 1010), 40, 10, 2, seed=nbl):
        x, z = np.meshgrid(np.arange(24) * 7.0, np.arange(24) * 7.0)
        shots.append(W.replace(sh, nbl=nbl, cfl_frac=0.99, src=np.array([[30.0, 40.0]]),
                               rec=np.stack([x.ravel(), z.ravel()], axis=1)))
    devs, dobs, _ = _device(shots)
    zero = [torch.zeros_like(d) for d in dobs]
    _, _, dsims, _ = _batch(devs, zero, 20 * devs[0].slot_bytes, 0.0, 0.0)
    for d, ds in zip(devs, dsims):
        data = d.forward()
        assert torch.count_nonzero(data[-1]) == data.shape[1] and torch.equal(data, ds)
