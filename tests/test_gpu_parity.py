"""GPU parity: the three library calls, through the C interface, against the
CPU reference on the same seeded inputs (bars in tests/parity.py)."""
import numpy as np
import pytest

from paper_2605_16867_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, params=["auto", "grouped"])
def scoring_layout(request):
    """Every test here runs twice: with the library choosing how a batch is scored
    (few pairs: pair by pair; many: through the table of its lengths), and always through the table."""
    parity.SMALL_BATCH_PAIRS = None if request.param == "auto" else 0
    yield
    parity.SMALL_BATCH_PAIRS = None


def report(name, rep):
    print(f"\n[{name}] " + " ".join(f"{k}={v}" for k, v in rep.items()), flush=True)


@pytest.mark.parametrize("name", ["tiny", "mid"])
def test_small_fleets_every_output(name):
    rep = parity.run_and_check(workloads.make_fleet(workloads.spec(name)))
    report(name, rep)


@pytest.mark.parametrize("scale", [2.0, 4.0, 16.0, 64.0])
def test_mid_fleet_decision_mix(scale):
    """Same shapes, looser SLOs, uneven occupancy, one idle instance: exercises
    the just-enough branch next to the fallback."""
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=scale, occupancy_jitter=True,
                                             seed=int(scale)))
    rep = parity.run_and_check(fl)
    report(f"mid x{scale}", rep)
    if scale <= 4.0:
        assert 0.02 < rep["route_feasible_frac"] < 1.0


def test_route_with_exclusions():
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=3.0, seed=5))
    rng = np.random.default_rng(1)
    ex = rng.integers(-1, fl.n_inst, len(fl.in_prompt)).astype(np.int32)
    report("exclude", parity.run_and_check(fl, exclude=ex))


# --------------------------------------------------------------------------- cached prefixes (Eq. 2's H)
@pytest.mark.parametrize("scale", [1.0, 2.0, 8.0])
def test_mid_fleet_with_cached_prefixes(scale):
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=scale, occupancy_jitter=True, seed=21))
    hits = workloads.cached_prefixes(fl, mean_hits=3.0, seed=1)
    rep = parity.run_and_check(fl, hits=hits)
    report(f"mid x{scale} + prefixes", rep)


def test_cached_prefixes_with_exclusions():
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=2.0, seed=22))
    hits = workloads.cached_prefixes(fl, mean_hits=4.0, seed=2)
    rng = np.random.default_rng(3)
    # half of the requests are barred from an instance they have a prefix on
    ex = np.full(len(fl.in_prompt), -1, dtype=np.int32)
    has = np.flatnonzero(np.diff(hits[0]) > 0)
    pick = has[rng.random(len(has)) < 0.5]
    ex[pick] = hits[1][hits[0][pick]]
    report("prefixes + exclude", parity.run_and_check(fl, exclude=ex, hits=hits))


# --------------------------------------------------------------------------- EMA-smoothed black-box status (Sec. 3.3)
@pytest.mark.parametrize("lam", [0.25, 1.0])
def test_mid_fleet_blended_with_black_box_status(lam):
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=2.0, occupancy_jitter=True, seed=31))
    rounds = workloads.observed_status(fl, rounds=3, seed=1)
    # the terms are not always observed together
    rounds.append((0.5, rounds[0][1], None, None))
    rep = parity.run_and_check(fl, blackbox=(rounds, lam))
    report(f"mid blend {lam}", rep)


def test_blend_with_prefixes_and_exclusions():
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=1.5, seed=32))
    hits = workloads.cached_prefixes(fl, mean_hits=3.0, seed=6)
    ex = np.random.default_rng(2).integers(-1, fl.n_inst, len(fl.in_prompt)).astype(np.int32)
    rep = parity.run_and_check(fl, exclude=ex, hits=hits, blackbox=(workloads.observed_status(fl, 2, seed=2), 0.6))
    report("mid blend 0.6 + prefixes + exclude", rep)


def test_observations_after_a_build_show_from_the_next_build_on():
    """Samples that arrive between a status build and a routing call change nothing the call
    sees: tables and capability order keep the estimates they were built with."""
    import torch
    dev = "cuda:0"
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=2.0, seed=33))
    d = parity.upload(fl, dev)
    rounds = workloads.observed_status(fl, 3, seed=6)
    f32t = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(dev)
    h = parity.make_handle(fl)
    for w, ow, op, od in rounds[:2]:
        h.gr_observe(w, f32t(ow), f32t(op), f32t(od))
    h.gr_set_blend(0.7)
    fin = torch.empty(len(fl.act_prompt), dtype=torch.float32, device=dev)
    n = len(fl.in_prompt)

    def route():
        inst = torch.full((n,), -7, dtype=torch.int32, device=dev)
        slack = torch.zeros(n, dtype=torch.float32, device=dev)
        h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], inst, slack)
        torch.cuda.synchronize()
        return inst.cpu().numpy(), slack.cpu().numpy()

    build = lambda: h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"],
                                      d["q_prompt"], d["q_len"], fin)
    build()
    w, ow, op, od = rounds[2]
    h.gr_observe(w, f32t(ow * 3.0), f32t(op * 3.0), f32t(od * 3.0))      # before the first routing call of this build
    a_inst, a_slack = route()
    h.gr_observe(w, f32t(ow), f32t(op * 0.2), f32t(od))                  # and between two routing calls
    b_inst, b_slack = route()
    assert np.array_equal(a_inst, b_inst) and np.array_equal(a_slack.view(np.uint32), b_slack.view(np.uint32))
    # the same fleet built after only the first two rounds routes the same way
    h2 = parity.make_handle(fl)
    for w2, ow2, op2, od2 in rounds[:2]:
        h2.gr_observe(w2, f32t(ow2), f32t(op2), f32t(od2))
    h2.gr_set_blend(0.7)
    fin2 = torch.empty_like(fin)
    h2.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin2)
    c_inst = torch.full((n,), -7, dtype=torch.int32, device=dev)
    c_slack = torch.zeros(n, dtype=torch.float32, device=dev)
    h2.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], c_inst, c_slack)
    torch.cuda.synchronize()
    assert np.array_equal(a_inst, c_inst.cpu().numpy()) and np.array_equal(a_slack.view(np.uint32), c_slack.cpu().numpy().view(np.uint32))
    # after a new build the samples do show
    build()
    e_inst, _ = route()
    assert (e_inst != a_inst).any()
    h.close(); h2.close()


def test_blend_zero_is_the_white_box_model_and_errors():
    from paper_2605_16867_amd import binding
    fl = workloads.make_fleet(workloads.spec("tiny"))
    rep0 = parity.run_and_check(fl)
    rep1 = parity.run_and_check(fl, blackbox=(workloads.observed_status(fl, 1, seed=4), 0.0))
    for k in ("finish_rel_err", "pair_T_rel_err", "route_differ", "route_ambiguous", "flag_frac", "flag_ambiguous",
              "migrate_differ", "migrate_ambiguous", "migrate_n"):
        assert rep0[k] == rep1[k], k
    h = parity.make_handle(fl)
    with pytest.raises(binding.GoodRouteError) as e:
        h.gr_set_blend(0.5)                       # nothing observed yet
    assert e.value.code == -4
    with pytest.raises(binding.GoodRouteError) as e:
        h.gr_set_blend(1.5)
    assert e.value.code == -1
    with pytest.raises(binding.GoodRouteError) as e:
        h.gr_observe(-0.1)
    assert e.value.code == -1
    h.gr_set_blend(0.0)
    h.close()


# --------------------------------------------------------------------------- routing with status feedback
@pytest.mark.parametrize("chunk", [1, 16, 100, 512])
def test_feedback_routing_mid_fleet(chunk):
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=3.0, occupancy_jitter=True, seed=41))
    rep = parity.run_feedback_and_check(fl, chunk, n_req=512)
    report(f"feedback chunk {chunk}", rep)
    assert rep["rounds"] == -(-512 // chunk)


def test_feedback_routing_spreads_the_herd():
    """Tight deadlines: one snapshot sends the whole batch to a few instances; feedback uses more."""
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=1.0, seed=42))
    snap = parity.run_feedback_and_check(fl, 512, n_req=512)
    fed = parity.run_feedback_and_check(fl, 8, n_req=512)
    report("feedback herd", {"snapshot_instances": snap["instances_used"], "feedback_instances": fed["instances_used"]})
    assert fed["instances_used"] >= snap["instances_used"]


def test_feedback_routing_large_fleet_with_exclusions():
    fl = workloads.make_fleet(workloads.spec("large", slo_scale=4.0, seed=43))
    ex = np.random.default_rng(4).integers(-1, fl.n_inst, 1024).astype(np.int32)
    rep = parity.run_feedback_and_check(fl, 128, n_req=1024, exclude=ex)
    report("feedback large", rep)


# --------------------------------------------------------------------------- batch cap (Sec. 3.1's memory bound)
@pytest.mark.parametrize("lo,hi", [(0.3, 1.2), (0.9, 1.0), (1.0, 1.0)])
def test_mid_fleet_with_batch_caps(lo, hi):
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=3.0, occupancy_jitter=True, seed=51))
    fl.batch_cap = workloads.batch_caps(fl, lo, hi, seed=1)
    rep = parity.run_and_check(fl)
    report(f"mid caps {lo}-{hi}", rep)


def test_batch_caps_with_everything_else():
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=2.0, seed=52))
    fl.batch_cap = workloads.batch_caps(fl, 0.4, 1.1, seed=2)
    hits = workloads.cached_prefixes(fl, mean_hits=3.0, seed=7)
    ex = np.random.default_rng(5).integers(-1, fl.n_inst, len(fl.in_prompt)).astype(np.int32)
    rep = parity.run_and_check(fl, exclude=ex, hits=hits, blackbox=(workloads.observed_status(fl, 2, seed=5), 0.4))
    report("mid caps + prefixes + exclude + blend", rep)


def test_tiny_fleet_with_queue_heavy_caps():
    fl = workloads.make_fleet(workloads.spec("tiny", n_queued=40, slo_scale=6.0, seed=53))
    for cap in (1, 7, 64, 103, 104, 105):
        fl.batch_cap = np.full(fl.n_inst, cap, dtype=np.int32)
        report(f"tiny cap {cap}", parity.run_and_check(fl))


@pytest.mark.parametrize("chunk,n_req", [(1, 200), (16, 512), (128, 1024), (700, 2100)])
def test_feedback_routing_with_batch_caps(chunk, n_req):
    """Under caps the order in which a chunk's requests queue up on an instance shows in every later
    estimate: it is the order of the batch, as in the reference."""
    fl = workloads.make_fleet(workloads.spec("mid", slo_scale=3.0, seed=54))
    fl.batch_cap = workloads.batch_caps(fl, 0.7, 1.05, seed=4)
    rep = parity.run_feedback_and_check(fl, chunk, n_req=n_req)
    report(f"feedback caps chunk {chunk}", rep)
