"""Batches decided through the table of runs (a group of lanes per request, and classes first in
large batches) against the pair-by-pair pass, which shares none of it: the same choices, slacks and
fallback bits, bit for bit.  Fleets at the sizes where a class fills, or just misses, whole runs;
lengths at the edges of the table's blocks; fleets full of exact ties; the exclusion of the very
instance a request would go to; a blend."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import CLASSES, fleet, rand_entries, solo

pytestmark = pytest.mark.gpu


def _route(call, d, sl, ex):
    import torch
    n = sl.stop - sl.start
    inst = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    slack = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda:0")
    fb = torch.full((n,), 9, dtype=torch.uint8, device="cuda:0")
    call(d["in_prompt"][sl], d["in_len"][sl], d["in_budget"][sl], inst, slack,
         exclude_inst=None if ex is None else ex[sl], out_fallback=fb)
    return inst, slack, fb


def _check(fl, blend=0.0, seed=0):
    import torch
    d = parity.upload(fl, "cuda:0")
    R, M = len(fl.in_prompt), len(fl.inst_class)
    h = parity.make_handle(fl)
    h.gr_set_small_batch_pairs(0)
    rng = np.random.default_rng(seed)
    if blend:
        obs = [torch.from_numpy(rng.uniform(lo, hi, M).astype(np.float32)).cuda() for lo, hi in
               ((0.0, 20.0), (1e-5, 2e-4), (0.02, 0.4))]
        h.gr_observe(1.0, *obs)
        h.gr_set_blend(blend)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device="cuda:0")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    whole = slice(0, R)
    first = _route(h.gr_score_route, d, whole, None)
    other = torch.from_numpy(rng.integers(-1, M, R).astype(np.int32)).cuda()
    feasible = 0
    for ex in (None, first[0], other):      # nobody excluded, everybody's own choice, somebody
        got = first if ex is None else _route(h.gr_score_route, d, whole, ex)
        step = 4096      # most requests of one call of gr_score_route_noalloc
        parts = [_route(h.gr_score_route_noalloc, d, slice(i, min(i + step, R)), ex) for i in range(0, R, step)]
        for k, a in enumerate(got):
            b = torch.cat([p[k] for p in parts])
            same = torch.eq(a, b) | (torch.isnan(a) & torch.isnan(b)) if k == 1 else torch.eq(a, b)
            assert bool(same.all()), f"output {k}: {int((~same).sum())} of {R} differ, first at {int(torch.nonzero(~same)[0])}"
        feasible += int((got[2] == 0).sum())
    assert h.gr_device_status() == 0
    h.close()
    return feasible / (3 * R)


def _fleet(n_inst, n_class, n_req, kind, n_len=None, seed=0):
    rng = np.random.default_rng([n_inst, n_class, n_req, seed])
    classes = [tuple(x * f for x in CLASSES[c % 3]) for c, f in enumerate(np.linspace(1.0, 1.7, n_class))]
    if kind == "idle":
        acts = [[] for _ in range(n_inst)]
    elif kind == "clones":
        some = [rand_entries(rng, int(n)) for n in rng.integers(1, 40, 5)]
        acts = [some[g % 5] for g in range(n_inst)]
    else:
        acts = [rand_entries(rng, int(n)) for n in rng.integers(0, 60, n_inst)]
    lens = np.clip(np.rint(rng.lognormal(5, 1, n_req)), 1, 4096).astype(np.int64)
    if n_len:
        lens = rng.choice(rng.permutation(np.arange(0, 4097))[:n_len], n_req)
    inc = np.stack([rng.integers(1, 2049, n_req), lens], 1)
    budgets = np.exp(rng.uniform(np.log(0.5), np.log(30), n_req)) * solo(inc[:, 0], inc[:, 1])
    budgets[::97] = np.inf
    budgets[1::97] = -1.0
    budgets[2::97] = np.nan
    return fleet(rng.integers(0, n_class, n_inst), acts, [[]] * n_inst, inc, budgets, classes=classes)


@pytest.mark.parametrize("kind", ["mixed", "clones", "idle"])
@pytest.mark.parametrize("n_inst,n_class", [(1, 1), (2, 2), (16, 1), (17, 1), (33, 3), (256, 3), (300, 20), (530, 2), (1100, 64)])
def test_runs_of_every_fill(n_inst, n_class, kind):
    _check(_fleet(n_inst, n_class, 1500, kind))


@pytest.mark.parametrize("n_len", [1, 255, 256, 257, 513])
def test_lengths_at_the_edges_of_a_block(n_len):
    assert 0.02 < _check(_fleet(100, 3, 3000, "mixed", n_len=n_len)) < 0.98


@pytest.mark.parametrize("blend", [0.5, 1.0])
@pytest.mark.parametrize("n_inst", [40, 700, 1100])
def test_blended(n_inst, blend):
    _check(_fleet(n_inst, 3, 1500, "mixed"), blend=blend)


@pytest.mark.parametrize("kind", ["mixed", "clones", "idle"])
@pytest.mark.parametrize("n_req,n_class", [((1 << 17) - 1, 3), (1 << 17, 3), ((1 << 17) + 37, 16), ((1 << 19) + 5, 4),
                                           ((1 << 19) - 1, 16), (1 << 19, 9), ((1 << 19) + 1, 16)])
def test_classes_first(n_req, n_class, kind):
    _check(_fleet(1300, n_class, n_req, kind))


# Least and next larger E of a class a rounding or a few apart (one queued prompt token is 2e-5 s), and prompts so long, or of the
# other sign, that their latencies fall together; as many classes as one piece, two, four and eight of 16 bytes hold.
@pytest.mark.parametrize("n_class,R", [(n, (1 << 17) + 1) for n in (1, 2, 3, 5, 8, 9, 16)] + [(n, (1 << 19) + 1) for n in (2, 9, 16)])
def test_classes_first_latencies_that_rounding_makes_equal(n_class, R):
    rng = np.random.default_rng(n_class)
    M = 1100
    classes = [tuple(x * f for x in CLASSES[c % 3]) for c, f in enumerate(np.linspace(1.0, 1.7, n_class))]
    some = [rand_entries(rng, int(n)) for n in rng.integers(1, 40, 5)]
    queued = [[(int(t), 4000)] if t else [] for t in rng.integers(0, 4, M)]
    inc = np.stack([rng.choice([1, 900, 2048, 1 << 15, 1 << 20, 1 << 24, 1 << 29, 0, -3, -(1 << 22)], R), rng.integers(0, 700, R)], 1)
    budgets = np.exp(rng.uniform(np.log(0.2), np.log(3), R)) * solo(np.abs(inc[:, 0]), inc[:, 1])
    _check(fleet(rng.integers(0, n_class, M), [some[g % 5] for g in range(M)], queued, inc, budgets, classes=classes))


@pytest.mark.parametrize("blend", [0.5, 1.0])
def test_classes_first_blended(blend):
    _check(_fleet(2200, 3, (1 << 17) + 3, "mixed"), blend=blend)
