"""The parity protocol of gpu_util on an oracle made for it: forcing one near-tie moves the oracle's own pass, and another decision, alike before, falls the
other way in its re-run."""
import numpy as np
import pytest

from gpu_util import gradient_parity


class Net:
    """Two ReLUs behind each other; the second one's z is `z` if the first one's near-tie is decided as here, else `moved`."""

    def __init__(self, moved):
        self.moved, self.runs = moved, 0

    def loss_and_grad(self, w, x, y, tie_break=None):
        self.runs += 1
        forced = [np.asarray((tie_break or {}).get(("relu", i), [-1, -1])) for i in (0, 1)]
        z = [np.array([3e-9, 1.0]), np.array([4e-9 if forced[0][0] < 0 else self.moved, 1.0])]
        active = [np.where(f < 0, v > 0, f).astype(np.int8) for f, v in zip(forced, z)]
        return 1.0, np.concatenate(active).astype(float), {("relu", 0): dict(z=z[0], active=active[0]), ("relu", 1): dict(z=z[1], active=active[1]),
                                                           "logits": np.ones(2)}


class Device:
    """Decides the first near-tie the other way, the second as the oracle's first run; off by 1e-8 elsewhere."""

    def worker_grad(self, p):
        return np.array([0.0, 1.0, 1.0, 1.0]), 1.0

    def workspace_tensor(self, p, kind, i):
        return np.ones(2) if kind == 2 else np.array([[0.0, 1 + 1e-8], [5e-9, 1 + 1e-8]][i])


def test_a_decision_that_turns_in_the_rerun():
    net, stats = Net(-6e-9), {}
    err, flips = gradient_parity(net, Device(), 0, None, None, None, stats)
    assert err == 0 and flips == 2 and net.runs == 3 and stats["grad_max_abs"] == 0


def test_one_that_turns_away_from_a_tie_is_refused():
    with pytest.raises(AssertionError, match="away from a tie"):
        gradient_parity(Net(-1e-6), Device(), 0, None, None, None)
