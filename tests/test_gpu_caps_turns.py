"""Capped instances with long queues, played turn by turn: one leaves and one comes, several leave and come at once
(equal lengths), room for many at the first turn, requests of one token, at every table size.  And without a queue, where nothing is played."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entries", [40, 64, 128, 256, 512, 1000, 2048])
@pytest.mark.parametrize("lengths", ["spread", "few", "mixed"])
def test_long_queues(entries, lengths):
    rng = np.random.default_rng([entries, len(lengths)])
    n_q = entries // 3
    A = entries - n_q
    caps = [1, max(A // 2, 1), A - 1, A, A + 1, A + n_q // 2, A + n_q - 1]
    acts, queued = [], []
    for k in range(len(caps)):
        e = rand_entries(rng, A)
        q = np.stack([rng.integers(1, 2049, n_q), rng.integers(1, 900, n_q)], 1)
        if lengths != "spread":
            few = [1, 2, 40, 41, 300] if lengths == "few" else [1, 40, 2000]
            some = rng.random(A) < (1.0 if lengths == "few" else 0.3)
            e[:, 2] = np.where(some, rng.choice(few, A), e[:, 2])
            some = rng.random(n_q) < (1.0 if lengths == "few" else 0.3)
            q[:, 1] = np.where(some, rng.choice(few, n_q), q[:, 1])
        acts.append(e)
        queued.append(q)
    inc = np.stack([rng.integers(128, 2049, 64), rng.integers(1, 3000, 64)], 1)
    fl = fleet(rng.integers(0, 3, len(caps)), acts, queued, inc, rng.uniform(1, 400, 64) * solo(inc[:, 0], inc[:, 1]))
    fl.batch_cap = np.asarray(caps, dtype=np.int32)
    parity.run_and_check(fl)


# (one running request, as many as the cap and one more or less; next to instances with a queue of one)
@pytest.mark.parametrize("entries", [1, 64, 65, 256, 512, 1024, 2048])
def test_without_a_queue(entries):
    rng = np.random.default_rng(entries)
    caps = [1, max(entries // 3, 1), max(entries - 1, 1), entries, entries + 1, entries + 5, 1, entries]
    acts = [rand_entries(rng, entries - (k >= 6)) for k in range(len(caps))]
    queued = [np.array([[700, 300]]) if k >= 6 else [] for k in range(len(caps))]
    inc = np.stack([rng.integers(128, 2049, 64), rng.integers(1, 3000, 64)], 1)
    fl = fleet(rng.integers(0, 3, len(caps)), acts, queued, inc, rng.uniform(1, 400, 64) * solo(inc[:, 0], inc[:, 1]))
    fl.batch_cap = np.asarray(caps, dtype=np.int32)
    parity.run_and_check(fl)
