"""out_T from the table pass: every latency equal, bit for bit, to the pair-by-pair pass, and the answers
equal to those of the same call without out_T; at the sizes where the layout changes (lanes per request,
instances per lane, Alg. 1 decided with the latencies or before them, more lengths than are turned into
rows at a time), for an array that starts anywhere."""
import numpy as np
import pytest

from tests import parity
from tests.test_gpu_runs import _fleet

pytestmark = pytest.mark.gpu


def _check(fl, shift=0):
    import torch
    d = parity.upload(fl, "cuda:0")
    R, M = len(fl.in_prompt), len(fl.inst_class)
    h = parity.make_handle(fl)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device="cuda:0")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    ex = torch.from_numpy(np.random.default_rng(M).integers(-1, M, R).astype(np.int32)).cuda()

    def route(pairs, with_T):
        h.gr_set_small_batch_pairs(pairs)
        inst = torch.full((R,), -7, dtype=torch.int32, device="cuda:0")
        slack = torch.full((R,), float("nan"), dtype=torch.float32, device="cuda:0")
        fb = torch.full((R,), 9, dtype=torch.uint8, device="cuda:0")
        T = torch.full((R * M + shift,), float("nan"), dtype=torch.float32, device="cuda:0")[shift:] if with_T else None
        h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], inst, slack, exclude_inst=ex, out_fallback=fb, out_T=T)
        torch.cuda.synchronize()
        return inst, slack, fb, T

    got, plain, direct = route(0, True), route(0, False), route(1 << 40, True)
    for other in (plain, direct):
        for a, b in zip(got, other):
            assert b is None or bool((torch.eq(a, b) | (torch.isnan(a) & torch.isnan(b))).all())
    assert not bool(torch.isnan(got[3]).any()) and h.gr_device_status() == 0
    h.close()


@pytest.mark.parametrize("n_inst", [1, 3, 15, 16, 17, 63, 64, 68, 127, 128, 129, 132, 511, 512, 516, 1025])
def test_fleet_sizes(n_inst):
    for shift in (0, 1):
        _check(_fleet(n_inst, min(n_inst, 3), 1003, "mixed"), shift)


@pytest.mark.parametrize("n_inst", [4500, 4501])
def test_more_lengths_than_are_turned_at_a_time(n_inst):
    fl = _fleet(n_inst, 3, 4096, "mixed")
    fl.in_len = np.random.default_rng(0).permutation(np.arange(1, 4097)).astype(np.int32)
    _check(fl)


@pytest.mark.parametrize("n_req", [1, 3, 4, 5, 7, 8, 9, 33, 127])
def test_requests_left_over(n_req):
    for n_inst in (40, 300):
        _check(_fleet(n_inst, 2, n_req, "clones"))
