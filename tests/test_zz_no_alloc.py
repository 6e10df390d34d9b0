"""gr_score_route_noalloc (the pair-by-pair pass for callers that want the same work queued whatever
the batch) against gr_score_route through the table pass, which shares none of it: the same inputs must
give the same instances, fallback bits and slacks bit for bit, on two calls in a row, the second
with a smaller batch, and on a second handle after the first is gone."""
import numpy as np
import pytest

from paper_2605_16867_amd import binding, workloads
from tests import parity

pytestmark = pytest.mark.gpu


def _route_both(h, d, n, exclude=None):
    import torch
    dev = "cuda:0"
    outs = []
    for call in (h.gr_score_route, h.gr_score_route_noalloc):
        inst = torch.full((n,), -7, dtype=torch.int32, device=dev)
        slack = torch.full((n,), float("nan"), dtype=torch.float32, device=dev)
        fb = torch.full((n,), 9, dtype=torch.uint8, device=dev)
        call(d["in_prompt"][:n], d["in_len"][:n], d["in_budget"][:n], inst, slack,
             exclude_inst=None if exclude is None else exclude[:n], out_fallback=fb)
        torch.cuda.synchronize()
        outs.append((inst.cpu().numpy(), slack.cpu().numpy(), fb.cpu().numpy()))
    return outs


def _same(a, b):
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[2], b[2])
    assert np.array_equal(a[1].view(np.uint32), b[1].view(np.uint32))


def test_noalloc_entry_point_matches_gr_score_route_on_two_calls_in_a_row():
    import torch
    dev = "cuda:0"
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=3.0, occupancy_jitter=True, seed=61))
    d = parity.upload(fl, dev)
    h = parity.make_handle(fl)
    h.gr_set_small_batch_pairs(0)                # gr_score_route through the table, whatever the batch
    fin = torch.empty(len(fl.act_prompt), dtype=torch.float32, device=dev)
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"],
                      d["q_len"], fin)
    n1, n2 = 4096, 1000
    ref1, got1 = _route_both(h, d, n1)
    _same(ref1, got1)
    ref2, got2 = _route_both(h, d, n2)            # smaller batch right after: nothing left over from the first
    _same(ref2, got2)
    assert np.array_equal(got2[0], got1[0][:n2])
    ex = torch.from_numpy(np.random.default_rng(0).integers(-1, fl.n_inst, n1).astype(np.int32)).to(dev)
    ref3, got3 = _route_both(h, d, 777, exclude=ex)
    _same(ref3, got3)
    # and against the CPU reference
    import oracle
    sim = oracle.simulate(fl)
    rep = {}
    parity.check_choices_all("noalloc", sim, fl.in_prompt[:n1], fl.in_len[:n1], fl.in_budget[:n1].astype(np.float64),
                             None, None, got1[0].astype(np.int64), got1[1], rep, fallback=got1[2])
    assert rep["noalloc_differ"] == 0
    # errors: too many requests, nothing built yet
    with pytest.raises(binding.GoodRouteError) as e:
        big = torch.zeros(4097, dtype=torch.int32, device=dev)
        h.gr_score_route_noalloc(big, big, big.float(), big.clone(), big.float())
    assert e.value.code == -2
    h.close()
    h2 = parity.make_handle(fl)
    with pytest.raises(binding.GoodRouteError) as e:
        h2.gr_score_route_noalloc(
            d["in_prompt"][:4], d["in_len"][:4], d["in_budget"][:4],
            torch.zeros(4, dtype=torch.int32, device=dev), torch.zeros(4, dtype=torch.float32, device=dev))
    assert e.value.code == -4
    # a second handle on the same GPU
    h2.gr_set_small_batch_pairs(0)
    h2.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"],
                       d["q_len"], fin)
    ref4, got4 = _route_both(h2, d, 300)
    _same(ref4, got4)
    assert np.array_equal(got4[0], got1[0][:300])
    assert h2.gr_device_status() == 0
    h2.close()
