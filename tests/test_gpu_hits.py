"""Cached prefixes: the short list of a request is shared by four lanes, unless every pair's latency is asked for, when one
thread takes it.  Both against each other bit for bit, with lists of every length around the four, instances named twice, not at
all or out of range, the excluded one and the one chosen without prefixes among them."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2605_16867_amd import workloads
from tests.parity import make_handle, upload

def up(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slo", [1.0, 8.0])
@pytest.mark.parametrize("blend", [0.0, 0.5])
@pytest.mark.parametrize("n_inst,n_req", [(5, 3), (40, 1025), (300, 4099)])
def test_lanes_against_one_thread(n_inst, n_req, blend, slo):
    sp = dataclasses.replace(workloads.spec("mid"), n_inst=n_inst, n_active=70, n_queued=3, n_incoming=n_req, slo_scale=slo, seed=11)
    fl = workloads.make_fleet(sp)
    rng = np.random.default_rng(n_req)
    h, d = make_handle(fl), upload(fl)
    if blend:
        for w, wait, prefill, decode in workloads.observed_status(fl, rounds=2, seed=3):
            h.gr_observe(w, up(wait), up(prefill), up(decode))
        h.gr_set_blend(blend)
    fin = torch.zeros(len(fl.act_prompt), device="cuda")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    out = lambda: (torch.zeros(n_req, dtype=torch.int32, device="cuda"), torch.zeros(n_req, device="cuda"),
                   torch.zeros(n_req, dtype=torch.uint8, device="cuda"))
    plain = out()
    h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], plain[0], plain[1], out_fallback=plain[2])
    first = plain[0].cpu().numpy()
    count = rng.choice([0, 1, 2, 3, 4, 5, 7, 8, 9, 17], n_req)
    off = np.concatenate([[0], np.cumsum(count)]).astype(np.int32)
    inst = rng.integers(-1, n_inst + 1, off[-1]).astype(np.int32)
    owner = np.repeat(np.arange(n_req), count)
    again = rng.random(off[-1]) < 0.2
    inst[again] = first[owner[again]]
    twice = np.flatnonzero((rng.random(off[-1]) < 0.3) & (np.arange(off[-1]) > 0))
    inst[twice] = inst[twice - 1]
    length = (rng.random(off[-1]) * 1.2 * fl.in_prompt[owner]).astype(np.int32)
    exclude = np.where(rng.random(n_req) < 0.5, rng.integers(0, n_inst, n_req), -1).astype(np.int32)
    hits = [up(off), up(inst), up(length)]
    got, want = out(), out()
    T = torch.zeros((n_req, n_inst), device="cuda")
    h.gr_score_route_cached(d["in_prompt"], d["in_len"], d["in_budget"], *hits, got[0], got[1], exclude_inst=up(exclude),
                            out_fallback=got[2])
    h.gr_score_route_cached(d["in_prompt"], d["in_len"], d["in_budget"], *hits, want[0], want[1], exclude_inst=up(exclude),
                            out_fallback=want[2], out_T=T)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    assert n_req < 100 or (got[0] != plain[0]).any()
