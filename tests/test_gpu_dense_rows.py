"""Tables with a row for every length, whose workgroups make the class order themselves, and the selection by four
lanes per request, against the pair-by-pair pass bit for bit: classes of 63 to 129 instances, fleets on both sides of the
most positions and of 16 and 32 runs, exact ties of d_g, lengths that include 0, large tables."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import CLASSES, fleet, rand_entries, solo
from tests.test_gpu_runs import _check, _fleet
from tests.test_gpu_scan_selection import _scan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["mixed", "clones", "idle"])
@pytest.mark.parametrize("n_inst,n_class,n_req", [(63, 1, 33000), (64, 1, 5000), (65, 1, 33000), (127, 1, 33000), (128, 1, 33000), (129, 1, 5000),
                                                  (240, 2, 33000), (300, 3, 40001), (330, 3, 5000), (400, 20, 33000), (70, 64, 33000)])
def test_routing(n_inst, n_class, n_req, kind):
    _check(_fleet(n_inst, n_class, n_req, kind))


@pytest.mark.parametrize("blend", [0.5, 1.0])
@pytest.mark.parametrize("n_inst,n_class", [(40, 1), (250, 3), (440, 4)])
def test_blended(n_inst, n_class, blend):
    _check(_fleet(n_inst, n_class, 33000, "mixed"), blend=blend)


@pytest.mark.parametrize("n_len", [1, 300, 4097])
def test_lengths_from_nothing(n_len):
    _check(_fleet(200, 3, 33000, "mixed", n_len=n_len))


@pytest.mark.parametrize("clones", [False, True])
@pytest.mark.parametrize("blend,obs", [(0.0, "many"), (0.5, "few"), (1.0, "odd")])
@pytest.mark.parametrize("late", ["all", "some"])
@pytest.mark.parametrize("n_inst,held,n_class", [(40, 1000, 1), (250, 140, 3), (430, 90, 4), (370, 400, 3), (60, 2000, 2)])
def test_scans(n_inst, held, n_class, late, blend, obs, clones):
    na, share, _ = _scan(n_inst, held, n_class, late, blend=blend, obs=obs, clones=clones)
    assert na >= 1 << 15 and share > 0.01


# positions (a class rounded up to 16s) times lengths: 288 x 4 097 = 1.2 M, 240 x 16 385 = 3.9 M, 288 x 16 385 = 4.7 M,
# 480 x 8 001 = 3.8 M, 480 x 16 385 = 7.9 M; the line is at 2^22 = 4.2 M
@pytest.mark.parametrize("n_inst,n_class,max_len,listed", [(250, 3, 4096, False), (200, 3, 16384, False), (250, 3, 16384, True),
                                                           (480, 6, 8000, False), (480, 6, 16384, True)])
def test_one_request_through_a_table_of_any_size(n_inst, n_class, max_len, listed):
    """A request with a cached prefix has a row of its own where a row for every length there may be would be a large
    table (the marks and the list are launched), and the answer is that of the pair-by-pair pass."""
    import torch
    rng = np.random.default_rng(n_inst)
    fl = fleet(np.arange(n_inst) % n_class, [rand_entries(rng, 20) for _ in range(n_inst)], [[]] * n_inst, np.array([[700, max_len]]),
               np.array([1.0]), classes=[tuple(x * (1 + c / 5) for x in CLASSES[0]) for c in range(n_class)], max_len=max_len)
    d = parity.upload(fl, "cuda:0")
    h = parity.make_handle(fl, max_requests=20000)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device="cuda:0")
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)
    z = lambda n, t, v=0: torch.full((n,), v, dtype=t, device="cuda:0")
    got, want = [[z(1, torch.int32, -7), z(1, torch.float32), z(1, torch.uint8, 9)] for _ in range(2)]
    req = [d[k] for k in ("in_prompt", "in_len", "in_budget")]
    h.gr_profile_enable(16)
    h.gr_score_route_cached(*req, z(2, torch.int32), z(0, torch.int32), z(0, torch.int32), got[0], got[1], out_fallback=got[2])
    ran = {k for k, (_, n) in h.gr_profile_read().items() if n}
    h.gr_score_route_noalloc(*req, want[0], want[1], out_fallback=want[2])
    assert ("k_mark<route>" in ran) == listed and "k_memo<route>" in ran
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    h.close()


@pytest.mark.parametrize("n_inst,n_class", [(2, 1), (64, 1), (65, 1), (128, 1), (250, 3), (440, 4)])
@pytest.mark.parametrize("step", [1e-17, 1e-13, 3e-12])
def test_next_decode_steps_closer_than_single_precision(n_inst, n_class, step):
    """d_g in the same order as its 64 bits have it where all, most or a few of a class are equal in single precision, some
    of them in full: instances hold as many requests each and differ by their contexts alone, which hardly cost anything."""
    rng = np.random.default_rng([n_inst, n_class])
    classes = [(2e-5, 0.012 * (1 + c / 10), 2e-4, step * (1 + c % 2)) for c in range(n_class)]
    ctx = rng.integers(1, 40, (n_inst, 3)) * 100
    acts = [np.stack([c, np.zeros(3, int), rng.integers(1, 400, 3)], 1) for c in ctx]
    d = np.array([classes[g % n_class][3] * float(c.sum()) + 0.0126 for g, c in enumerate(ctx)])
    assert n_inst < 60 or len(np.unique(d.astype(np.float32))) < len(np.unique(d))
    n_req = 33000
    inc = np.stack([rng.integers(1, 2049, n_req), np.clip(np.rint(rng.lognormal(5, 1, n_req)), 1, 4096)], 1)
    budgets = np.exp(rng.uniform(np.log(0.5), np.log(30), n_req)) * solo(inc[:, 0], inc[:, 1])
    share = _check(fleet(np.arange(n_inst) % n_class, acts, [[]] * n_inst, inc, budgets, classes=classes))
    assert share > 0.02


@pytest.mark.parametrize("late", ["all", "some"])
@pytest.mark.parametrize("n_inst,held,n_class", [(470, 300, 5), (458, 300, 6), (476, 300, 5)])      # 32 runs, a row per length
def test_large_scans_at_the_most_runs(n_inst, held, n_class, late):
    na, share, _ = _scan(n_inst, held, n_class, late)
    assert na >= 1 << 17 and share > 0.01
