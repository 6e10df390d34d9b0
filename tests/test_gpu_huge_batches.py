"""Batches of so many requests that one launch does not hold all threads of a kernel: the same few requests
over and over must be answered the same way from the first to the last."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu

PERIOD = 61


def _handle(n_inst, n_class, n, seed=0):
    import torch
    rng = np.random.default_rng([n_inst, n_class, seed])
    inc = np.stack([rng.integers(1, 2049, PERIOD), rng.integers(1, 600, PERIOD)], 1)
    fl = fleet(np.arange(n_inst) % n_class, [rand_entries(rng, int(k)) for k in rng.integers(0, 40, n_inst)], [[]] * n_inst, inc,
               np.exp(rng.uniform(np.log(0.6), np.log(10), PERIOD)) * solo(inc[:, 0], inc[:, 1]),
               classes=[(2e-5 * f, 0.012 * f, 2e-4 * f, 2e-8 * f) for f in np.linspace(1, 3, n_class)])
    d = parity.upload(fl, "cuda:0")
    h = parity.make_handle(fl, max_requests=n)
    h.gr_set_small_batch_pairs(0)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device="cuda:0")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    return h, d


def _route(h, d, n, T=False):
    import torch
    over = lambda x: x.repeat(-(-n // PERIOD))[:n].contiguous()
    inst = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    slack = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda:0")
    out_T = torch.full((n * h.n_inst,), float("nan"), dtype=torch.float32, device="cuda:0") if T else None
    h.gr_score_route(over(d["in_prompt"]), over(d["in_len"]), over(d["in_budget"]), inst, slack, out_T=out_T)
    torch.cuda.synchronize()
    return inst, slack, out_T


def _periodic(x, first):
    whole = x.numel() // first.numel() * first.numel()
    assert bool((x[:whole].view(-1, first.numel()) == first).all())
    assert bool((x[whole:] == first[:x.numel() - whole]).all())


@pytest.mark.parametrize("n_inst,n_class", [(3, 2), (40, 17)])
def test_more_requests_than_a_launch_has_groups_of_lanes(n_inst, n_class):
    n = (1 << 28) + 5
    h, d = _handle(n_inst, n_class, n)
    first = _route(h, d, PERIOD)
    assert len(first[0].unique()) > 1
    got = _route(h, d, n)
    for a, b in zip(got[:2], first[:2]):
        _periodic(a, b)
    h.close()


@pytest.mark.parametrize("n_inst", [2, 17])
def test_more_requests_than_a_launch_has_workgroups(n_inst):
    n = (1 << 24) + 5
    h, d = _handle(n_inst, 2, n)
    first = _route(h, d, PERIOD, T=True)
    got = _route(h, d, n, T=True)
    for a, b in zip(got, first):
        _periodic(a, b)
    h.close()
