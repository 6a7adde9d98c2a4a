"""3-D grids whose rows end inside a float4: the row's last lane reads and writes pad columns."""
import numpy as np
import pytest

from tests.helpers import gpu_side, has_gpu, oracle_side, rel_l2, small_3d

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


@pytest.mark.parametrize("n,order", [((17, 20, 19), 4), ((18, 21, 18), 16), ((19, 18, 20), 8), ((15, 19, 18), 8)],
                         ids=["33", "34", "35", "31"])
def test_rows_that_end_inside_a_float4(n, order):
    """Padded row lengths of 4k+1..3 (the layer is 8 cells): data, final state and a Revolve
    gradient within the solver tests' tolerances of the oracle, and bit-identical whether the
    workspace starts as zeros or as NaN (checkpoint slots then hold NaN beside their rows)."""
    import torch
    shot = small_3d(n=n, nt=60, order=order)
    S, _ = oracle_side(shot)
    St, _ = oracle_side(shot, "true")
    fw = S.forward(want_traj=True)
    res = fw["data"] - St.forward()["data"]
    gref = S.gradient_full(fw["traj"], res)
    G, _ = gpu_side(shot)
    rt = torch.as_tensor(res.astype(np.float32), device="cuda")
    out = []
    for fill in (0, 0xFF):
        ws = G.workspace(1, 4 * G.slot_bytes)
        G._ws.fill_(fill)
        data, state = G.forward(want_state=True)
        G._ws.fill_(fill)
        g, st = G.gradient(rt, 4 * G.slot_bytes)
        out.append((data, state, g))
        del ws
    assert all(torch.equal(a, b) for a, b in zip(*out))
    assert rel_l2(out[0][0].cpu().numpy(), fw["data"]) <= 1e-5
    assert rel_l2(out[0][1][0].cpu().numpy(), fw["traj"][-1]) <= 1e-5
    assert rel_l2(out[0][2].cpu().numpy(), gref) <= 1e-4
