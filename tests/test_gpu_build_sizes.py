"""Instances that hold far less than the handle has room for: the build picks how many words to sort
per instance, at the sizes where the choice changes, for every table size; and chunks of feedback
routing of up to a wave, which join their instances inside the build."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu


def _fleet(sizes, n_req, seed):
    rng = np.random.default_rng(seed)
    acts, queued = [], []
    for s in sizes:
        q = min(int(rng.integers(0, 4)), s)
        acts.append(rand_entries(rng, s - q))
        queued.append(np.stack([rng.integers(128, 2049, q), rng.integers(1, 900, q)], 1))
    inc = np.stack([rng.integers(128, 2049, n_req), rng.integers(1, 3000, n_req)], 1)
    fl = fleet(rng.integers(0, 3, len(sizes)), acts, queued, inc, rng.uniform(1, 200, n_req) * solo(inc[:, 0], inc[:, 1]))
    fl.act_budget = rng.uniform(1.0, 800.0, len(fl.act_prompt)).astype(np.float32)
    return fl


@pytest.mark.parametrize("cap", [128, 256, 512, 1024, 2048])
def test_words_by_what_an_instance_holds(cap):
    edges = [cap // 4 - 1, cap // 4, cap // 4 + 1, cap // 2 - 1, cap // 2, cap // 2 + 1]
    fl = _fleet([cap] + edges + [0, 1, 2, 3] + [cap // 8] * 6, 100, cap)
    parity.run_and_check(fl)


@pytest.mark.parametrize("chunk", [1, 63, 64, 65])
def test_chunks_that_join_in_the_build(chunk):
    sizes = [30, 120, 60, 0, 125, 127, 64, 3]
    fl = _fleet(sizes, 200, chunk)
    parity.run_feedback_and_check(fl, chunk)
