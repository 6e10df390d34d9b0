"""Tables with a row for every length, whose workgroups make the class order themselves, and the selection by four
lanes per request, against the pair-by-pair pass bit for bit: classes of 63 to 129 instances, fleets on both sides of the
most positions and of 16 and 32 runs, exact ties of d_g, lengths that include 0, large tables."""
import numpy as np
import pytest

from tests.fleets import fleet, solo
from tests.test_gpu_runs import _check, _fleet
from tests.test_gpu_scan_selection import _scan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["mixed", "clones", "idle"])
@pytest.mark.parametrize("n_inst,n_class,n_req", [(63, 1, 33000), (64, 1, 5000), (65, 1, 33000), (127, 1, 33000), (128, 1, 33000), (129, 1, 5000),
                                                  (240, 2, 33000), (300, 3, 40001), (330, 3, 5000), (400, 20, 33000), (70, 64, 33000)])
def test_routing(n_inst, n_class, n_req, kind):
    _check(_fleet(n_inst, n_class, n_req, kind))


@pytest.mark.parametrize("blend", [0.5, 1.0])
@pytest.mark.parametrize("n_inst,n_class", [(40, 1), (250, 3), (440, 4)])
def test_blended(n_inst, n_class, blend):
    _check(_fleet(n_inst, n_class, 33000, "mixed"), blend=blend)


@pytest.mark.parametrize("n_len", [1, 300, 4097])
def test_lengths_from_nothing(n_len):
    _check(_fleet(200, 3, 33000, "mixed", n_len=n_len))


@pytest.mark.parametrize("clones", [False, True])
@pytest.mark.parametrize("blend,obs", [(0.0, "many"), (0.5, "few"), (1.0, "odd")])
@pytest.mark.parametrize("late", ["all", "some"])
@pytest.mark.parametrize("n_inst,held,n_class", [(40, 1000, 1), (250, 140, 3), (430, 90, 4), (370, 400, 3), (60, 2000, 2)])
def test_scans(n_inst, held, n_class, late, blend, obs, clones):
    na, share, _ = _scan(n_inst, held, n_class, late, blend=blend, obs=obs, clones=clones)
    assert na >= 1 << 15 and share > 0.01


@pytest.mark.parametrize("n_inst,n_class", [(2, 1), (64, 1), (65, 1), (128, 1), (250, 3), (440, 4)])
@pytest.mark.parametrize("step", [1e-17, 1e-13, 3e-12])
def test_next_decode_steps_closer_than_single_precision(n_inst, n_class, step):
    """d_g in the same order as its 64 bits have it where all, most or a few of a class are equal in single precision, some
    of them in full: instances hold as many requests each and differ by their contexts alone, which hardly cost anything."""
    rng = np.random.default_rng([n_inst, n_class])
    classes = [(2e-5, 0.012 * (1 + c / 10), 2e-4, step * (1 + c % 2)) for c in range(n_class)]
    ctx = rng.integers(1, 40, (n_inst, 3)) * 100
    acts = [np.stack([c, np.zeros(3, int), rng.integers(1, 400, 3)], 1) for c in ctx]
    d = np.array([classes[g % n_class][3] * float(c.sum()) + 0.0126 for g, c in enumerate(ctx)])
    assert n_inst < 60 or len(np.unique(d.astype(np.float32))) < len(np.unique(d))
    n_req = 33000
    inc = np.stack([rng.integers(1, 2049, n_req), np.clip(np.rint(rng.lognormal(5, 1, n_req)), 1, 4096)], 1)
    budgets = np.exp(rng.uniform(np.log(0.5), np.log(30), n_req)) * solo(inc[:, 0], inc[:, 1])
    share = _check(fleet(np.arange(n_inst) % n_class, acts, [[]] * n_inst, inc, budgets, classes=classes))
    assert share > 0.02
