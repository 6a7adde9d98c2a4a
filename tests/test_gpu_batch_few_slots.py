"""2-D batches whose checkpoint memory holds one state or a few, so that most steps are
recomputation (a program has far more groups of steps than actions): the solo call's bits."""
import pytest

from tests.helpers import has_gpu
from tests.test_gpu_batch import _batch, _device, _shots

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


@pytest.mark.parametrize("slots,nt", [(0, 100), (1, 300), (2, 300)])
@pytest.mark.parametrize("tol", [0.0, 1e-4], ids=["plain", "compressed"])
def test_few_slots_match_solo(slots, nt, tol):
    """slots: uncompressed states in the budget (with none, each state is recomputed from the
    start); a ratio of 1 plans as many compressed ones."""
    import torch
    devs, dobs, _ = _device(_shots((37, 34), nt, 8, 2, seed=5 + slots))
    budget = int((slots + 0.5) * devs[0].slot_bytes)
    hint = 1.0 if tol > 0 else 0.0
    phis, grads, dsims, sts = _batch(devs, dobs, budget, tol, hint)
    for i, d in enumerate(devs):
        phi, g, st, ds = d.misfit_gradient(dobs[i], budget, tol, ratio_hint=hint, want_dsim=True)
        assert st["slots"] == slots + 1
        assert sts[i]["slots"] == st["slots"] and sts[i]["advances"] == st["advances"]
        assert phis[i] == phi and torch.equal(dsims[i], ds) and torch.equal(grads[i], g)
