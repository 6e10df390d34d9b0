"""Tables with a row for every length, whose workgroups make the class order themselves, and the selection by four
lanes per request, against the pair-by-pair pass bit for bit: classes of 63 to 129 instances, fleets on both sides of the
most positions and of 16 and 32 runs, exact ties of d_g, lengths that include 0, large tables."""
import numpy as np
import pytest

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
