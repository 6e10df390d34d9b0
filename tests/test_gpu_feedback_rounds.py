"""Feedback routing with a launch per decision round (chunks of up to 64 requests, up to 512 instances, tables of at least 128
entries) against the same rounds through the table of lengths, a scoring pass and a rebuild each, bit for bit: answers and the
tables left behind, for every size of table, instances on both sides of a wave's share and of the limits, the first rebuild taking
every instance or only the chosen ones."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2605_16867_amd import workloads
from tests.parity import make_handle, upload

pytestmark = pytest.mark.gpu


def _route(fl, chunk, n, entries, pairs, blend, exclude, stale):
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    h, d = make_handle(fl, max_entries=entries), upload(fl)
    if pairs is not None:
        h.gr_set_small_batch_pairs(pairs)
    if blend:
        for w, wait, prefill, decode in workloads.observed_status(fl, rounds=2, seed=3):
            h.gr_observe(w, dev(wait), dev(prefill), dev(decode))
    if not stale:
        h.gr_set_blend(blend)
    fin = torch.zeros(max(len(fl.act_prompt), 1), device="cuda")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    if stale:       # (the tables are of another weight: the first rebuild takes every instance)
        h.gr_set_blend(blend)
    out = [torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.zeros(n, device="cuda"),
           torch.zeros(n, dtype=torch.uint8, device="cuda")]
    ex = None if exclude is None else dev(exclude)
    req = [d[k][:n] for k in ("in_prompt", "in_len", "in_budget")]
    for _ in range(2):      # (the second call goes on from what the first one has routed)
        h.gr_route_feedback(chunk, *req, out[0], out[1], exclude_inst=ex, out_fallback=out[2])
    after = [torch.zeros_like(x) for x in out]
    h.gr_score_route(*req, after[0], after[1], out_fallback=after[2])
    assert h.gr_device_status() == 0
    return out + after


@pytest.mark.parametrize("n_inst,held,entries", [
    (1, 70, 128), (2, 1, 200), (3, 30, 250), (63, 100, 300), (64, 300, 512), (65, 120, 400), (255, 200, 700), (256, 520, 2048),
    (257, 40, 1024), (300, 1000, 1500), (511, 60, 128), (512, 100, 513), (513, 100, 300), (40, 20, 64)])
@pytest.mark.parametrize("chunk,n", [(1, 5), (7, 50), (63, 130), (64, 128), (64, 3), (65, 150)])
def test_by_round(n_inst, held, entries, chunk, n):
    n = min(n, (entries - held - 3) // 2)
    variant = n_inst + chunk
    sp = dataclasses.replace(workloads.spec("mid"), n_inst=n_inst, n_active=held, n_queued=min(3, held // 10), n_incoming=n,
                             slo_scale=(1.0, 4.0, 16.0)[variant % 3], seed=variant)
    fl = workloads.make_fleet(sp)
    rng = np.random.default_rng(variant)
    exclude = np.where(rng.random(n) < 0.5, rng.integers(0, n_inst, n), -1).astype(np.int32) if variant % 2 else None
    blend, stale = (0.0, 0.5, 1.0)[variant % 3], variant % 5 < 2
    got = _route(fl, chunk, n, entries, None, blend, exclude, stale)
    want = _route(fl, chunk, n, entries, 0, blend, exclude, stale)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("who", ["all", "some"])
@pytest.mark.parametrize("bits", [0x7fc00000, 0x7fffffff, -1, -0x400000])
def test_observations_that_are_no_numbers(bits, who):
    """Latencies that are NaNs, of every sign and with every bit set, have their place in the order of the pair-by-pair pass:
    one instance takes the request.  Tables of 64 entries (a pass and a rebuild per round) against tables of 128."""
    sp = dataclasses.replace(workloads.spec("mid"), n_inst=9, n_active=20, n_queued=2, n_incoming=21, seed=5)
    fl = workloads.make_fleet(sp)
    nan = torch.tensor([bits], dtype=torch.int32).view(torch.float32).cuda().expand(9).contiguous()
    one = torch.from_numpy(np.linspace(1e-4, 2e-4, 9).astype(np.float32)).cuda()
    seen = []
    for entries in (64, 128):
        h, d = make_handle(fl, max_entries=entries), upload(fl)
        wait = one * 1e4
        if who == "some":
            wait[2:5] = nan[2:5]
        else:
            wait = nan
        h.gr_observe(1.0, wait, one, one * 500)
        h.gr_set_blend(0.5)
        fin = torch.zeros(len(fl.act_prompt), device="cuda")
        h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
        out = [torch.full((21,), -7, dtype=torch.int32, device="cuda"), torch.zeros(21, device="cuda"),
               torch.zeros(21, dtype=torch.uint8, device="cuda")]
        ex = torch.arange(21, dtype=torch.int32, device="cuda") % 9
        h.gr_route_feedback(5, *[d[k] for k in ("in_prompt", "in_len", "in_budget")], out[0], out[1], exclude_inst=ex, out_fallback=out[2])
        seen.append([x.cpu().numpy() for x in out])
        h.close()
    assert (seen[0][0] >= 0).all()
    for a, b in zip(*seen):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
