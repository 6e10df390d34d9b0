"""Risk scans and routing batches that are scored pair by pair because they are small, against the same calls
through the table, bit for bit: fleets on both sides of each number of lanes per request, batches up to the
rule's line and one past it, instances that nobody can use (infinite observations), flags that no instance sets."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu

LINE = 1 << 19       # pairs


def _fleet(n_inst, held, n_in, seed):
    rng = np.random.default_rng([n_inst, held, seed])
    sizes = np.full(n_inst, held)
    if n_inst > 2:
        sizes[rng.integers(0, n_inst, 2)] = [0, held // 2]
    acts = [rand_entries(rng, int(n)) for n in sizes]
    all_ = np.concatenate(acts)
    budget = np.exp(rng.uniform(np.log(0.5), np.log(40), len(all_))) * solo(all_[:, 0] + all_[:, 1], all_[:, 2])
    budget[::97], budget[1::97], budget[2::97] = np.inf, -1.0, np.nan
    inc = np.stack([rng.integers(128, 2049, n_in), rng.choice([1, 3, 50, 400, 2000], n_in)], 1)
    return fleet(rng.integers(0, 3, n_inst), acts, [[(700, 30)] if g % 3 == 0 else [] for g in range(n_inst)], inc,
                 np.exp(rng.uniform(np.log(0.5), np.log(60), n_in)) * solo(inc[:, 0], inc[:, 1]), act_budget=budget)


def _both_ways(fl, off, obs):
    """Outputs of a scan, a routing call and a second scan: by the library's own rule, through the table."""
    import torch
    d = parity.upload(fl, "cuda:0")
    M, na, R = len(fl.inst_class), len(fl.act_prompt), len(fl.in_prompt)
    rng = np.random.default_rng(M)
    seen = []
    samples = [rng.uniform(0, 20, M), rng.uniform(1e-5, 2e-4, M), rng.uniform(0.02, 0.4, M)]
    if obs == "some infinite":
        samples[0][::3] = np.inf
    if obs == "all infinite":
        samples[0][:] = np.inf
    flags0 = torch.from_numpy((rng.random(na) < 0.5).astype(np.uint8) * 3).cuda()
    for pairs in (None, 0):
        h = parity.make_handle(fl, max_entries=int(np.diff(fl.act_off).max()) + 1)
        if pairs is not None:
            h.gr_set_small_batch_pairs(pairs)
        if obs:
            h.gr_observe(1.0, *[torch.from_numpy(x.astype(np.float32)).cuda() for x in samples])
            h.gr_set_blend(0.5)
        z = lambda n, t, v=0: torch.full((n,), v, dtype=t, device="cuda:0")
        flag, fin, tgt, tsl, nfl = flags0.clone(), z(na, torch.float32), z(na, torch.int32, -7), z(na, torch.float32, 7), z(1, torch.int32)
        inst, slack, fb = z(R, torch.int32, -7), z(R, torch.float32, 7), z(R, torch.uint8, 9)
        got = []
        for o in (d["act_off"], off, d["act_off"]):
            h.gr_risk_scan(o, d["act_prompt"], d["act_gen"], d["act_rem_refreshed"], d["q_off"], d["q_prompt"], d["q_len"],
                           d["act_budget"], flag, fin, tgt, tsl, nfl)
            h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], inst, slack, out_fallback=fb)
            got += [x.clone() for x in (flag, fin, tgt, tsl, nfl, inst, slack, fb)]
        torch.cuda.synchronize()
        late = flag != 0
        assert int(nfl.item()) == int(late.sum()) and bool((tgt[~late] == -1).all())
        seen.append([x.cpu().numpy() for x in got])
        h.close()
    for k, (a, b) in enumerate(zip(*seen)):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), f"output {k % 8} of round {k // 8}"


@pytest.mark.parametrize("obs", [None, "some infinite", "all infinite"])
@pytest.mark.parametrize("n_inst,held", [(1, 1), (1, 700), (4, 64), (16, 513), (17, 100), (32, 512), (33, 90), (64, 128), (65, 60),
                                         (512, 2), (513, 1), (720, 1)])
def test_small_scans(n_inst, held, obs):
    import torch
    n_in = min(LINE // max(n_inst, 16), 20000)
    fl = _fleet(n_inst, held, n_in + n_inst % 2, len(obs or ""))      # (one request past the line on odd fleets)
    na = len(fl.act_prompt)
    assert na * max(n_inst, 16) <= LINE
    off = np.clip(fl.act_off.astype(np.int64), na // 7, na - na // 7).astype(np.int32)      # entries in nobody's slice
    _both_ways(fl, torch.from_numpy(off).cuda(), obs)


@pytest.mark.parametrize("n", [1 << 14, (1 << 14) + 1])
def test_the_line(n):
    """32 instances: 2^14 running requests are scored pair by pair, one more through the table."""
    rng = np.random.default_rng(n)
    acts = [rand_entries(rng, 512 + (n - (1 << 14) if g == 0 else 0)) for g in range(32)]
    all_ = np.concatenate(acts)
    assert len(all_) == n
    fl = fleet(rng.integers(0, 3, 32), acts, [[]] * 32, np.ones((8, 2)), np.ones(8),
               act_budget=rng.uniform(0.5, 20, n) * solo(all_[:, 0] + all_[:, 1], all_[:, 2]))
    import torch
    _both_ways(fl, torch.from_numpy(fl.act_off).cuda(), None)


@pytest.mark.parametrize("n,pairs,inst", [(1, None, 0), (2048, None, 0), (2049, None, -1), (8193, None, -1), (2048, 0, -1), (2049, 1 << 19, 0)])
def test_infinite_latencies_by_size(n, pairs, inst):
    """64 instances whose every latency is infinite: a small batch goes to the lowest index (and any batch scored pair by pair that
    the caller has set the size of), a larger one nowhere, gr_score_route_noalloc always somewhere."""
    import torch
    fl = _fleet(64, 2, 10000, 1)
    d = parity.upload(fl, "cuda:0")
    h = parity.make_handle(fl)
    if pairs is not None:
        h.gr_set_small_batch_pairs(pairs)
    obs = torch.full((64,), float("inf"), device="cuda:0")
    h.gr_observe(1.0, obs, obs, obs)
    h.gr_set_blend(0.5)
    z = lambda n, t, v=0: torch.full((n,), v, dtype=t, device="cuda:0")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"],
                      z(len(fl.act_prompt), torch.float32))
    got, fb, other = z(n, torch.int32, -7), z(n, torch.uint8, 9), z(n, torch.int32, -7)
    slack = z(n, torch.float32)
    req = [d[k][:n] for k in ("in_prompt", "in_len", "in_budget")]
    h.gr_score_route(*req, got, slack, out_fallback=fb)
    assert bool((got == inst).all()) and bool((fb == 1).all())
    assert bool((slack == (0 if inst < 0 else -float("inf"))).all())
    if n <= 4096:
        h.gr_score_route_noalloc(*req, other, slack)
        assert bool((other == 0).all())
    if inst == 0:
        h.gr_route_feedback(64, *[x[:64] for x in req], other[:64], slack[:64])
        assert bool((other[:64] == 0).all())
    h.close()
