"""Large batches by every way of deciding them (the classes first, the lines that can be least first, a lane or a
group of lanes per request, a list for what is left) against the pair-by-pair pass, bit for bit: risk
scans (every target and slack, the request's own instance excluded), and batches whose prompts lie on and next to
the ends of the ranges that lines are looked up for.  Ties, idle instances, late requests of any share,
observations of one or two values, infinite ones."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import CLASSES, fleet, rand_entries, solo
from tests.test_gpu_runs import _fleet, _route

pytestmark = pytest.mark.gpu

PART = 4096      # most requests of one call of gr_score_route_noalloc


def _observe(h, M, rng, kind):
    import torch
    few = lambda lo, hi: rng.choice(np.linspace(lo, hi, 2), M)
    many = lambda lo, hi: rng.uniform(lo, hi, M)
    draw = few if kind == "few" else many
    obs = [draw(0.0, 20.0), draw(1e-5, 2e-4), draw(0.02, 0.4)]
    if kind == "odd":
        obs[0][::7] = np.inf
        obs[1][1::7] = np.inf
        obs[2][2::7] = -0.01
    h.gr_observe(1.0, *[torch.from_numpy(x.astype(np.float32)).cuda() for x in obs])


def _scan(n_inst, held, n_class, late, blend=0.0, obs="many", clones=False, seed=0, total=None):
    import torch
    rng = np.random.default_rng([n_inst, held, n_class, seed])
    classes = [tuple(x * f for x in CLASSES[c % 3]) for c, f in enumerate(np.linspace(1.0, 1.7, n_class))]
    sizes = np.full(n_inst, held)
    sizes[rng.integers(0, n_inst, 3)] = [0, 1, held - 1]
    if total is not None:
        sizes[:] = held
        sizes[:n_inst * held - total] -= 1
    some = rand_entries(rng, held)
    acts = [some[:n] if clones else rand_entries(rng, int(n)) for n in sizes]
    all_ = np.concatenate(acts)
    na = len(all_)
    alone = solo(all_[:, 0] + all_[:, 1], all_[:, 2])
    lo, hi = {"all": (0.2, 1.5), "some": (1.0, 60.0), "few": (10.0, 400.0)}[late]
    budget = np.exp(rng.uniform(np.log(lo), np.log(hi), na)) * alone
    budget[::97], budget[1::97], budget[2::97] = np.inf, -1.0, np.nan
    fl = fleet(rng.integers(0, n_class, n_inst), acts, [[]] * n_inst, np.ones((PART, 2)), np.ones(PART), classes=classes, act_budget=budget)
    d = parity.upload(fl, "cuda:0")
    h = parity.make_handle(fl)
    if blend:
        _observe(h, n_inst, rng, obs)
        h.gr_set_blend(blend)
    z = lambda n, t, v=0: torch.full((n,), v, dtype=t, device="cuda:0")
    flag, fin, tgt, tsl, nfl = z(na, torch.uint8, 9), z(na, torch.float32), z(na, torch.int32, -7), z(na, torch.float32, 7), z(1, torch.int32)
    for _ in range(2):       # (the second scan finds what the first one has left)
        h.gr_risk_scan(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem_refreshed"], d["q_off"], d["q_prompt"], d["q_len"],
                       d["act_budget"], flag, fin, tgt, tsl, nfl)
        own = torch.repeat_interleave(torch.arange(n_inst, dtype=torch.int32, device="cuda:0"), torch.from_numpy(sizes).cuda())
        off = flag == 0
        assert bool((tgt[off] == -1).all()) and bool((tsl[off] == 0).all()) and int(nfl.item()) == int((~off).sum())
        idx = torch.nonzero(~off).flatten()
        c0, ln, bud, own = [x[idx].contiguous() for x in (d["act_prompt"] + d["act_gen"], d["act_rem_refreshed"], d["act_budget"], own)]
        feasible = 0
        for i in range(0, len(idx), PART):
            s = slice(i, i + PART)
            n = len(idx[s])
            inst, slack, fb = z(n, torch.int32, -7), z(n, torch.float32), z(n, torch.uint8)
            h.gr_score_route_noalloc(c0[s].contiguous(), ln[s].contiguous(), bud[s].contiguous(), inst, slack,
                                     exclude_inst=own[s].contiguous(), out_fallback=fb)
            same = (tgt[idx[s]] == inst) & ((tsl[idx[s]] == slack) | (torch.isnan(tsl[idx[s]]) & torch.isnan(slack)))
            assert bool(same.all()), f"{int((~same).sum())} of {n} differ, first at {int(torch.nonzero(~same)[0])}"
            feasible += int((fb == 0).sum())
    assert h.gr_device_status() == 0
    h.close()
    return na, len(idx) / na, feasible / max(len(idx), 1)


# the classes first: 2^17 requests and more, 2^18 and more
@pytest.mark.parametrize("clones", [False, True])
@pytest.mark.parametrize("late", ["all", "some"])
@pytest.mark.parametrize("n_inst,held,n_class", [(520, 257, 3), (1100, 121, 16), (530, 1001, 4)])
def test_scan_classes_first(n_inst, held, n_class, late, clones):
    na, share, _ = _scan(n_inst, held, n_class, late, clones=clones)
    assert na >= 1 << 17 and share > 0.01


# the classes first, by four lanes a request up to 2^18 of them, by one from there on; up to 8 classes, and more
@pytest.mark.parametrize("late", ["all", "some"])
@pytest.mark.parametrize("n_class", [3, 9, 16])
@pytest.mark.parametrize("total", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1])
def test_scan_classes_first_by_lanes(total, n_class, late):
    na, share, _ = _scan(1100, 239, n_class, late, total=total)
    assert na == total and share > 0.01


# over the runs (less than 3 * 2^16 requests), and the lines first (more than 80 runs, less than 2^19 requests)
@pytest.mark.parametrize("obs", ["many", "few", "odd"])
@pytest.mark.parametrize("late", ["all", "some"])
@pytest.mark.parametrize("n_inst,held", [(1400, 99), (2000, 101)])
def test_scan_lines_first(n_inst, held, late, obs):
    na, share, _ = _scan(n_inst, held, 3, late, blend=0.5, obs=obs)
    assert (1 << 17) <= na < (1 << 19) and (na >= 3 << 16) == (held == 101) and share > 0.01


# the lines first, a lane per request and a list of the rest (2^19 requests and more)
@pytest.mark.parametrize("blend,obs", [(0.5, "many"), (1.0, "many"), (1.0, "few"), (0.5, "odd")])
@pytest.mark.parametrize("late", ["all", "some", "few"])
@pytest.mark.parametrize("n_inst,held", [(530, 1001), (2100, 251)])
def test_scan_lines_and_list(n_inst, held, late, blend, obs):
    na, share, _ = _scan(n_inst, held, 3, late, blend=blend, obs=obs)
    assert na >= (1 << 19) and share > 0.001


# more runs than a wave reads at once (320), and than the list's kernel keeps in LDS (1 024)
@pytest.mark.parametrize("late", ["all", "few"])
@pytest.mark.parametrize("n_inst,held", [(5300, 100), (17000, 31)])
def test_scan_of_wide_fleets(n_inst, held, late):
    na, share, _ = _scan(n_inst, held, 3, late, blend=1.0)
    assert na >= (1 << 19) and share > 0.001


@pytest.mark.parametrize("clones", [False, True])
@pytest.mark.parametrize("late", ["all", "some"])
def test_scan_of_more_classes_than_are_looked_at_first(late, clones):
    na, share, _ = _scan(560, 950, 17, late, clones=clones)
    assert na >= (1 << 19) and share > 0.001


@pytest.mark.parametrize("obs", ["many", "few", "odd"])
@pytest.mark.parametrize("blend", [0.5, 1.0])
def test_prompts_at_the_ends_of_the_ranges(blend, obs):
    import torch
    fl = _fleet(1500, 3, (1 << 17) + 11, "mixed")
    rng = np.random.default_rng(5)
    R, M = len(fl.in_prompt), 1500
    ends = np.array([1024, 4096, 16384, 131072])
    fl.in_prompt = rng.choice(np.concatenate([ends - 1, ends, ends + 1, [1, 2, 1 << 20, 1 << 24]]), R).astype(np.int32)
    fl.in_budget[::3] = (np.exp(rng.uniform(np.log(0.5), np.log(30), len(fl.in_budget[::3]))) * solo(fl.in_prompt[::3], fl.in_len[::3])).astype(np.float32)
    d = parity.upload(fl, "cuda:0")
    h = parity.make_handle(fl)
    _observe(h, M, rng, obs)
    h.gr_set_blend(blend)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device="cuda:0")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    first = _route(h.gr_score_route, d, slice(0, R), None)
    for ex in (None, first[0]):
        got = first if ex is None else _route(h.gr_score_route, d, slice(0, R), ex)
        parts = [_route(h.gr_score_route_noalloc, d, slice(i, min(i + PART, R)), ex) for i in range(0, R, PART)]
        for k, a in enumerate(got):
            b = torch.cat([p[k] for p in parts])
            assert bool((torch.eq(a, b) | (torch.isnan(a) & torch.isnan(b)) if k == 1 else torch.eq(a, b)).all()), f"output {k}"
    h.close()
