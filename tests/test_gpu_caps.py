"""More requests running than the batch cap allows, with a queue behind them: the departures before
the first admission in closed form, at every table size, with the cap next to the number that
run and with many requests of one length (they leave together)."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entries", [64, 128, 256, 512, 1024, 2048])
def test_overfull_batches_with_a_queue(entries):
    rng = np.random.default_rng(entries)
    n_q = 5
    A = entries - n_q
    caps = [1, 2, A // 2, A - 1, A, A + 1, A + n_q, A + n_q + 1]
    acts, queued = [], []
    for k in range(len(caps)):
        e = rand_entries(rng, A)
        if k % 2:
            e[:, 2] = rng.choice([1, 40, 41, 700], A)
        acts.append(e)
        queued.append(np.stack([rng.integers(128, 2049, n_q), rng.integers(1, 900, n_q)], 1))
    inc = np.stack([rng.integers(128, 2049, 64), rng.integers(1, 3000, 64)], 1)
    fl = fleet(rng.integers(0, 3, len(caps)), acts, queued, inc, rng.uniform(1, 400, 64) * solo(inc[:, 0], inc[:, 1]))
    fl.batch_cap = np.asarray(caps, dtype=np.int32)
    fl.act_budget = rng.uniform(1.0, 2000.0, len(fl.act_prompt)).astype(np.float32)
    rep = parity.run_and_check(fl)
    assert 0 < rep["flag_frac"] < 1
