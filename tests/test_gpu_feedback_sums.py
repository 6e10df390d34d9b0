"""Feedback routing that adds what has come to the sums of the tables as they were built last, against the same rounds through
the table of lengths and a rebuild each, bit for bit: instances whose lists are taken in several times, that run out of
room, that have requests from an earlier call, and lengths out of range."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2605_16867_amd import workloads
from tests.fleets import fleet
from tests.parity import make_handle, upload

pytestmark = pytest.mark.gpu


def _route(fl, chunk, entries, pairs, blend, lens):
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    h, d = make_handle(fl, max_entries=entries), upload(fl)
    if pairs is not None:
        h.gr_set_small_batch_pairs(pairs)
    if blend:
        for w, wait, prefill, decode in workloads.observed_status(fl, rounds=2, seed=3):
            h.gr_observe(w, dev(wait), dev(prefill), dev(decode))
        h.gr_set_blend(blend)
    fin = torch.zeros(len(fl.act_prompt), device="cuda")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    R = len(fl.in_prompt)
    out = []
    for n in (R, R // 2):      # (the second call goes on from what the first one has routed)
        got = [torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.zeros(n, device="cuda"),
               torch.zeros(n, dtype=torch.uint8, device="cuda")]
        h.gr_route_feedback(chunk, d["in_prompt"][:n], dev(lens)[:n], d["in_budget"][:n], got[0], got[1], out_fallback=got[2])
        out += got
    after = [torch.full((R,), -7, dtype=torch.int32, device="cuda"), torch.zeros(R, device="cuda"),
             torch.zeros(R, dtype=torch.uint8, device="cuda"), torch.zeros(R, fl.n_inst, device="cuda")]
    h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], after[0], after[1], out_fallback=after[2], out_T=after[3])
    status = h.gr_device_status()
    h.close()
    return out + after, status


@pytest.mark.parametrize("n_inst,held,entries,chunk,n", [
    (4, 20, 400, 1, 150), (5, 100, 512, 7, 300), (3, 60, 128, 8, 300), (9, 120, 1024, 8, 900), (33, 20, 2048, 8, 600), (40, 90, 130, 9, 200),
    (40, 90, 130, 10, 200), (40, 90, 130, 11, 200), (256, 30, 140, 64, 400), (320, 30, 140, 64, 400), (321, 30, 140, 64, 300), (512, 20, 128, 40, 300)])
@pytest.mark.parametrize("blend,odd_lengths", [(0.0, False), (0.5, True), (1.0, False)])
def test_same_as_rebuilt(n_inst, held, entries, chunk, n, blend, odd_lengths):
    sp = dataclasses.replace(workloads.spec("mid"), n_inst=n_inst, n_active=held, n_queued=held // 10, n_incoming=n,
                             slo_scale=(1.0, 4.0, 16.0)[(n_inst + chunk) % 3], occupancy_jitter=True, seed=n_inst + chunk)
    fl = workloads.make_fleet(sp)
    rng = np.random.default_rng(chunk)
    lens = fl.in_len.copy()
    if odd_lengths:
        lens[rng.random(n) < 0.2] = rng.choice([0, -3, sp.max_len, sp.max_len + 5])
    got, status = _route(fl, chunk, entries, None, blend, lens)
    want, want_status = _route(fl, chunk, entries, 0, blend, lens)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    assert status == want_status


@pytest.mark.parametrize("entries,sent", [(128, 128), (128, 129), (128, 131), (128, 132), (256, 256), (256, 257), (256, 263)])
def test_dropped_requests_are_reported(entries, sent):
    """Idle instances whose room is the whole table.  All requests but the last go to one of them (the most loaded instance is
    the least capable one that still serves in time), the last one elsewhere: what is beyond the room is only
    seen by the build at the end, which nothing joins."""
    n = sent + 1
    fl = fleet([0, 1, 2, 0, 1], [[]] * 5, [[]] * 5, [(100 + i % 7, 50 + i % 5) for i in range(n)], np.full(n, 1e9))
    got = []
    for pairs in (None, 0):
        h, d = make_handle(fl, max_entries=entries), upload(fl)
        if pairs is not None:
            h.gr_set_small_batch_pairs(pairs)
        out = [torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.zeros(n, device="cuda")]
        h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"],
                          torch.zeros(0, device="cuda"))
        exclude = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        exclude[-1] = 2
        h.gr_route_feedback(1, d["in_prompt"], d["in_len"], d["in_budget"], *out, exclude_inst=exclude)
        got.append((*out, h.gr_device_status()))
        h.close()
    assert torch.all(got[0][0][:-1] == 2) and got[0][0][-1] != 2
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert got[0][2] == got[1][2] == (2 if sent > entries else 0)      # (GR_DEV_ENTRIES_DROPPED)
