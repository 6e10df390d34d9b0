"""Device memory of a handle: parts that only some handles can use are not reserved by the others."""
import numpy as np
import pytest
import torch

from paper_2605_16867_amd import binding
from tests.fleets import CLASSES

pytestmark = pytest.mark.gpu


def _held(n_inst, n_class, entries, max_len, max_requests, handles=1):
    """Bytes that a handle takes (of several, as small allocations share a block)."""
    coef = [np.array([CLASSES[c % 3][i] for c in range(n_class)]) for i in range(4)]

    def make():
        return binding.Fleet(*coef, np.arange(n_inst, dtype=np.int32) % n_class, entries, max_len, max_requests)

    make().close()      # (what the runtime itself takes for the first one)
    before = torch.cuda.mem_get_info()[0]
    hs = [make() for _ in range(handles)]
    held = before - torch.cuda.mem_get_info()[0]
    for h in hs:
        h.close()
    return held / handles


def test_minima_by_row_only_where_classes_may_come_first():
    """4 096 instances of six classes, a row for each of 16 385 lengths either way: 16 640 rows of 272 minima more from 131 072 requests on, and none for more classes than a group has lanes."""
    rows, runs = 16640, 272
    few, many = (_held(4096, 6, 64, 16384, n) for n in (131071, 131072))
    assert many - few >= 0.9 * rows * runs * 4
    few, many = (_held(4096, 17, 64, 16384, n) for n in (131071, 131072))
    assert many - few < 0.1 * rows * runs * 4


def test_feedback_sums_only_where_waves_share_an_instance():
    """512 instances: 65 to 128 entries take (50 * 128 + 1 200) * 512 bytes that up to 64 entries do not, besides the tables,
    whose 18 bytes an entry and 8 a request double."""
    small, large = _held(512, 3, 64, 64, 1, 32), _held(512, 3, 128, 64, 1, 32)
    assert large - small >= 0.9 * 512 * ((50 * 128 + 1200) + 64 * 26)
