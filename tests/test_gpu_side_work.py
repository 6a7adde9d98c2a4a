"""3-D steps that inject and gather in their own launch, at the edges of that choice: points in
one to four planes, in more (a launch of their own), at the tops and bottoms of chunks, several
sources, and two sources that share grid points (which keeps the source's launch of its own)."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_side, has_gpu, oracle_side, rel_l2, small_3d

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


def _shot(rec_z, src, nt=50, order=8, time_order=2):
    """A small shot with receivers at random (x, y) on the given depths (in cells), on and
    between the nodes of a line, and sources at the given places (in cells)."""
    shot = small_3d(n=(37, 34, 33), nt=nt, order=order)
    rng = np.random.default_rng(len(rec_z) + 10 * len(src))
    rec = np.array([[x, y, z] for z in rec_z for x, y in rng.uniform(0, 33, size=(1200 // len(rec_z), 2))])
    rec[::3, :2] = np.round(rec[::3, :2])
    return W.replace(shot, rec=rec * 10.0, src=np.array(src, dtype=float) * 10.0,
                     vel_true=(shot.vel * 1.02).astype(np.float32))


CASES = {
    "one_plane": ([3.0], [[18.0, 17.0, 3.0]]),
    "two_planes": ([3.5], [[18.3, 17.6, 3.4]]),
    "four_planes": ([0.0, 7.0, 20.0, 32.0], [[18.0, 17.0, 3.0], [9.0, 5.0, 30.0], [4.5, 9.5, 12.0]]),
    "five_planes": ([0.0, 7.0, 20.0, 25.0, 32.0], [[5.0 * i, 17.0, 6.0 * i] for i in range(1, 6)]),
    "shared_points": ([2.0], [[18.25, 17.5, 3.5], [18.75, 17.25, 3.25]]),
}


@pytest.mark.parametrize("time_order", [2, 4])
@pytest.mark.parametrize("name", list(CASES))
def test_injection_and_gather_planes(name, time_order):
    import torch
    shot = _shot(*CASES[name])
    S, _ = oracle_side(shot, time_order=time_order)
    St, _ = oracle_side(shot, "true", time_order=time_order)
    fw = S.forward(want_traj=True)
    res = fw["data"] - St.forward()["data"]
    gref = S.gradient_full(fw["traj"], res)
    G, _ = gpu_side(shot, time_order=time_order)
    data, state = G.forward(want_state=True)
    assert rel_l2(data.cpu().numpy(), fw["data"]) <= 1e-5
    assert rel_l2(state[0].cpu().numpy(), fw["traj"][-1]) <= 1e-5
    rt = torch.as_tensor(res.astype(np.float32), device="cuda")
    g, _ = G.gradient(rt, G.slot_bytes * 6)
    full, _ = G.gradient(rt, G.slot_bytes * shot.nt)
    assert torch.equal(g, full)
    assert rel_l2(g.cpu().numpy(), gref) <= 1e-4
    # the transpose of the source path, whose steps carry no gradient
    ref = S.adjoint_src(res)
    assert rel_l2(G.adjoint_src(rt).cpu().numpy(), ref) <= 1e-4
