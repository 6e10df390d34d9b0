"""Batches scored pair by pair, whose lanes read each other's instances' words: every table size, fleets that fill no group
of lanes, and the blends (at weight 1 every segment of an instance is alike and none is searched for), against the
table pass bit for bit, every pair's latency among the outputs."""
import dataclasses

import numpy as np
import pytest

from paper_2605_16867_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weight", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("cap", [64, 128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("n_inst", [3, 18, 67, 131])
def test_same_as_the_table(n_inst, cap, weight):
    import torch
    dev = "cuda:0"
    fl = workloads.make_fleet(dataclasses.replace(workloads.spec("mid"), n_inst=n_inst, n_active=cap - cap // 8, n_queued=cap // 16,
                                                  n_incoming=201, slo_scale=4.0, occupancy_jitter=True, seed=cap + n_inst))
    d = parity.upload(fl, dev)
    h = parity.make_handle(fl, max_entries=cap)
    if weight:
        for w, wait, prefill, decode in workloads.observed_status(fl, rounds=2, seed=1):
            h.gr_observe(w, *(torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in (wait, prefill, decode)))
        h.gr_set_blend(weight)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device=dev)
    R = len(fl.in_prompt)
    ex = torch.from_numpy((np.arange(R) % (n_inst + 1) - 1).astype(np.int32)).to(dev)
    got = []
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    for pairs in (1 << 40, 0):
        h.gr_set_small_batch_pairs(pairs)
        out = [torch.full((R,), -7, dtype=torch.int32, device=dev), torch.zeros(R, dtype=torch.float32, device=dev),
               torch.full((R,), 9, dtype=torch.uint8, device=dev), torch.zeros(R, n_inst, dtype=torch.float32, device=dev)]
        h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], out[0], out[1], exclude_inst=ex, out_fallback=out[2],
                         out_T=out[3])
        torch.cuda.synchronize()
        got.append([x.cpu().numpy() for x in out])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    assert 0.0 < np.mean(got[0][2] == 0) and np.all(got[0][3] > 0)
    assert h.gr_device_status() == 0
    h.close()


# (the library's own choice next to the table: below, at and above the largest batch that is scored pair by pair)
@pytest.mark.parametrize("n_inst,n", [(16, 49152), (20, 39321), (20, 39322), (33, 15887), (64, 12288), (64, 12289), (100, 6144), (100, 6145), (130, 4096), (700, 1117), (1030, 722)])
def test_largest_small_batches(n_inst, n):
    import torch
    dev = "cuda:0"
    fl = workloads.make_fleet(dataclasses.replace(workloads.spec("mid"), n_inst=n_inst, n_active=40, n_queued=3, n_incoming=n,
                                                  slo_scale=4.0, occupancy_jitter=True, seed=n))
    d = parity.upload(fl, dev)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device=dev)
    got = []
    for pairs in (None, 0):
        h = parity.make_handle(fl)
        if pairs is not None:
            h.gr_set_small_batch_pairs(pairs)
        out = [torch.full((n,), -7, dtype=torch.int32, device=dev), torch.zeros(n, dtype=torch.float32, device=dev),
               torch.full((n,), 9, dtype=torch.uint8, device=dev)]
        h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
        h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], out[0], out[1], out_fallback=out[2])
        torch.cuda.synchronize()
        got.append([x.cpu().numpy() for x in out])
        h.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
