"""The smoother calls of a training step: small batches ask for the partition kernel."""

import pytest
import torch

from paper_2604_00048_amd import learned


class Asked(Exception):
    pass


@pytest.mark.parametrize("P,staged", [(1, False), (64, False), (1024, False), (1025, True), (4096, True)])
@pytest.mark.parametrize("form", [learned.Learned, learned.LearnedScalar])
def test_training_batches_choose_the_kernel_of_their_size(form, P, staged, monkeypatch):
    asked = {}

    def solve(x, w, lam, d, P, **kw):
        asked["solve"] = kw.get("staged", True)
        return x, None

    def backward(w, lam, z, g, d, P, need_x, **kw):
        asked["backward"] = kw.get("staged", True)
        raise Asked

    monkeypatch.setattr(learned.whs, "whs_solve", solve)
    monkeypatch.setattr(learned.whs, "whs_backward", backward)
    monkeypatch.setattr(learned.net, "mse", lambda *a, **k: None)
    f = object.__new__(form)
    f.device, f.sd = torch.device("cpu"), 1.0
    monkeypatch.setattr(f, "weights", lambda *a, **k: (None, None))
    t = torch.zeros(1)
    batch = learned.Batch(P, t, t, t, t, 1, None, 1)
    with pytest.raises(Asked):
        f.train_step(batch, 0.1, *([] if form is learned.Learned else [1.0]))
    assert asked == {"solve": staged, "backward": staged}
