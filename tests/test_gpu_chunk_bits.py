"""A 3-D step's bits do not depend on how its planes are split over workgroups: a model mirrored
in z, whose chunks meet other planes, gives the mirrored wavefield."""
import numpy as np
import pytest

from tests.helpers import has_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


@pytest.mark.parametrize("n,order", [((24, 24, 59), 8), ((41, 30, 45), 4), ((56, 56, 41), 12)])
def test_mirrored_in_z(n, order):
    """The waves ahead of the front reach every corner of the layer within the run.  The mirrored
    sums take z's two neighbours in the other order, which rounds alike."""
    import torch
    import paper_1810_05268_amd as P
    from paper_1810_05268_amd.shot import DeviceShot
    nbl, nt, h = 12, 60, (10.0, 10.0, 10.0)
    dt = 0.8 * P.cfl_dt(3, h, order, 3700.0)
    rng = np.random.default_rng(order)
    vel = rng.uniform(2500.0, 3500.0, size=tuple(v + 2 * nbl for v in reversed(n))).astype(np.float32)
    q = np.sin(np.arange(nt) * 0.3).astype(np.float32)
    src = np.array([[(n[0] // 2) * 10.0, (n[1] // 2) * 10.0, 50.0]])
    rec = np.array([[10.0, 10.0, 20.0]])
    flip = np.array([1.0, 1.0, -1.0]), np.array([0.0, 0.0, (n[2] - 1) * 10.0])
    out = []
    for v, s, r in ((vel, src, rec), (vel[::-1], flip[1] + flip[0] * src, flip[1] + flip[0] * rec)):
        S = DeviceShot(3, n, h, nbl, order, nt, dt, 3700.0, np.ascontiguousarray(v), q, s, r)
        out.append(S.forward(want_state=True))
    (d0, u0), (d1, u1) = out
    assert torch.count_nonzero(u0[0]) > 0.9 * u0[0].numel()
    assert torch.equal(d0, d1) and torch.equal(u0, torch.flip(u1, dims=[1]))
