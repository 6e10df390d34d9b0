"""Batches scored pair by pair, at the sizes where the layout changes: lanes per request (up to 16,
64, 512, 1 024 instances, several instances per lane, several workgroups per request), and every
table size of the two-step search (splitters, then one stride), with lengths on and next to the
table's own."""
import numpy as np
import pytest

import oracle
from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu


def _route_all(fl, max_entries, exclude=None):
    """The batch through gr_score_route pair by pair, through gr_score_route_noalloc and through the table
    pass: equal bit for bit, every choice against the reference."""
    import torch
    dev = "cuda:0"
    d = parity.upload(fl, dev)
    h = parity.make_handle(fl, max_entries=max_entries)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device=dev)
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    R = len(fl.in_prompt)
    ex = None if exclude is None else torch.from_numpy(exclude).to(dev)
    got = []
    for call, pairs in ((h.gr_score_route, 1 << 40), (h.gr_score_route_noalloc, 1 << 40), (h.gr_score_route, 0)):
        h.gr_set_small_batch_pairs(pairs)
        inst = torch.full((R,), -7, dtype=torch.int32, device=dev)
        slack = torch.full((R,), float("nan"), dtype=torch.float32, device=dev)
        fb = torch.full((R,), 9, dtype=torch.uint8, device=dev)
        call(d["in_prompt"], d["in_len"], d["in_budget"], inst, slack, exclude_inst=ex, out_fallback=fb)
        torch.cuda.synchronize()
        got.append((inst.cpu().numpy(), slack.cpu().numpy(), fb.cpu().numpy()))
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
    rep = {}
    parity.check_choices_all("direct", oracle.simulate(fl), fl.in_prompt, fl.in_len, fl.in_budget.astype(np.float64),
                             exclude, None, got[0][0].astype(np.int64), got[0][1], rep, fallback=got[0][2])
    assert rep["direct_differ"] <= 0.001 * R
    assert h.gr_device_status() == 0
    h.close()
    return rep


@pytest.mark.parametrize("n_inst", [1, 15, 16, 17, 63, 64, 65, 256, 257, 512, 513, 1024, 1025, 2047, 4095, 4096, 4097, 8193])
def test_fleet_sizes(n_inst):
    rng = np.random.default_rng(n_inst)
    acts = [rand_entries(rng, int(n)) for n in rng.integers(0, 9, n_inst)]
    n = 37
    inc = np.stack([rng.integers(128, 2049, n), rng.choice([1, 3, 50, 400, 2000], n)], 1)
    fl = fleet(rng.integers(0, 3, n_inst), acts, [[]] * n_inst, inc, rng.uniform(0.8, 6, n) * solo(inc[:, 0], inc[:, 1]))
    for me in (8, 1024):
        _route_all(fl, me)
        _route_all(fl, me, exclude=rng.integers(-1, n_inst, n).astype(np.int32))


@pytest.mark.parametrize("n", [3276, 3277, 4096])
def test_more_parts_than_there_is_room_for(n):
    """Five parts of 4 096 instances per request: 16 384 selections are kept at most, and beyond that one
    workgroup takes all instances of a request."""
    rng = np.random.default_rng(n)
    acts = [rand_entries(rng, int(k)) for k in rng.integers(0, 3, 17000)]
    inc = np.stack([rng.integers(128, 2049, n), rng.choice([1, 3, 50, 400, 2000], n)], 1)
    _route_all(fleet(rng.integers(0, 3, 17000), acts, [[]] * 17000, inc, rng.uniform(0.8, 6, n) * solo(inc[:, 0], inc[:, 1])), 8)


@pytest.mark.parametrize("cap", [64, 128, 256, 512, 1024, 2048])
def test_table_sizes(cap):
    rng = np.random.default_rng(cap)
    sizes = [0, 1, 7, 8, 9, cap // 2, cap - 1, cap]
    acts = []
    for s in sizes:
        e = rand_entries(rng, s)
        if s:
            e[:, 2] = rng.choice([1, 2, 30, 31, 500, 4095, 4096], s) if s % 2 else rng.integers(1, 4097, s)
        acts.append(e)
    own = np.unique(np.concatenate([a[:, 2] for a in acts if len(a)]))
    lens = np.clip(np.concatenate([rng.choice(own, 150) + k for k in (-1, 0, 1)] + [[1, 4096]]), 1, 4096).astype(np.int64)
    inc = np.stack([rng.integers(128, 2049, len(lens)), lens], 1)
    fl = fleet(rng.integers(0, 3, len(sizes)), acts, [[]] * len(sizes), inc,
               np.exp(rng.uniform(np.log(0.4), np.log(60), len(lens))) * solo(inc[:, 0], inc[:, 1]))
    rep = _route_all(fl, cap)
    assert 0.02 < rep["direct_feasible_frac"] < 1.0
