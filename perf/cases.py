"""The work that a user of this library has it do, as cases that can be timed.

A serving proxy keeps a fleet handle, refreshes the status of its instances, routes what has
arrived since, and re-checks the running requests from time to time.  A case is one such call
or round of calls on a synthetic fleet (``workloads``), inputs and outputs in device memory.

Plain values of a case:

  call      what one pass does
            "step"     gr_build_status + gr_score_route + gr_risk_scan: a whole control interval
            "refresh"  gr_build_status + gr_score_route: the status is refreshed, then a batch is routed
            "route"    gr_score_route on a status that stands
            "cached"   gr_build_status + gr_score_route_cached (prompts with cached prefixes)
            "feedback" gr_build_status + gr_route_feedback, `chunk` requests per decision round
            "status"   gr_build_status with every output
            "scan"     gr_risk_scan
  inst, held, queued, incoming   instances; running and queued requests per instance; requests routed
  classes   GPU classes of the fleet: 2 or 3 (the named classes), 6 (spaced geometrically)
  tail      True: Pareto decode lengths up to 16 384 and lognormal prompts; False: lognormal
            decode lengths up to 4 096 and uniform prompts
  slo       scale of the deadlines: 1 as the recipe draws them (most requests find nobody who meets
            theirs), larger ones let the just-enough choice decide
  ragged    instances hold between a quarter and all of `held`, one of them nothing
  exclude   half of the requests may not go to one instance (a retry goes elsewhere)
  caps      the decode batch of every instance is bounded
  blend     weight of the smoothed black-box status
  chunk     see "feedback"; 0 elsewhere
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2605_16867_amd import binding, workloads


def _case(call, inst, held, queued, incoming, classes=3, tail=False, slo=1.0, ragged=False, exclude=False,
          caps=False, blend=0.0, chunk=0):
    return dict(call=call, inst=inst, held=held, queued=queued, incoming=incoming, classes=classes, tail=tail,
                slo=slo, ragged=ragged, exclude=exclude, caps=caps, blend=blend, chunk=chunk)


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)

    return [
        # four instances, sixteen arrivals: launches and host time are all there is
        named("tiny_step", "step", 4, 64, 8, 16, classes=2),
        # the paper's own order: the status is refreshed, one arriving request is routed
        named("one_arrival", "refresh", 256, 512, 0, 1),
        # the arrivals of a moment on a standing status, estimated from observed figures alone
        named("arrivals_48", "route", 1024, 1000, 0, 48, blend=1.0),
        # a rack: a control interval of the mid-sized fleet
        named("mid_step", "step", 32, 256, 32, 4096),
        # the large fleet, deadlines that some instances can meet
        named("large_step", "step", 256, 512, 0, 65536, slo=4.0),
        # nothing round: uneven instances, queues, an odd number of everything, loose deadlines, retries
        named("ragged_loose", "refresh", 777, 301, 9, 20011, slo=16.0, ragged=True, exclude=True),
        # periodic re-check of a million running requests
        named("migrate_scan", "scan", 1024, 1000, 0, 0),
        # status refresh of the largest fleet, every output asked for
        named("heavy_status", "status", 4096, 512, 0, 0, classes=6, tail=True),
        # a quarter of a million arrivals on the largest fleet, long tails
        named("heavy_route", "refresh", 4096, 512, 0, 262144, classes=6, tail=True),
        # periodic re-check of the largest fleet
        named("heavy_scan", "scan", 4096, 512, 0, 0, classes=6, tail=True),
        # agentic sessions: prefixes cached on a few instances, batches bounded by memory
        named("cached_capped", "cached", 1024, 200, 40, 32768, slo=2.0, caps=True),
        # decisions that see the ones before them, 64 requests at a time
        named("feedback_64", "feedback", 256, 512, 0, 2048, chunk=64),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call = rng.choice(["step", "refresh", "refresh", "route", "cached", "feedback", "status", "scan", "scan"])
    inst = _log_int(rng, 4, 4096 if call != "feedback" else 512)
    held = _log_int(rng, 16, min(1000, (1 << 21) // inst))
    queued = rng.choice([0, 0, max(1, held // 8)])
    incoming = _log_int(rng, 1, 262144)
    chunk = 0
    if call in ("status", "scan"):
        incoming = 0
    elif call == "feedback":
        chunk = _log_int(rng, 1, 512)
        incoming = min(chunk * rng.randint(2, 16) + rng.randint(0, chunk), 4096)
    elif call == "step":
        incoming = min(incoming, 65536)
        inst = min(inst, 2048)
    return _case(call, inst, held, queued, incoming, classes=rng.choice([2, 3, 6]), tail=rng.random() < 0.4,
                 slo=rng.choice([1.0, 1.0, 2.0, 4.0, 16.0]), ragged=rng.random() < 0.4,
                 exclude=call in ("refresh", "route", "cached", "feedback") and rng.random() < 0.3,
                 caps=rng.random() < 0.15, blend=rng.choice([0.0, 0.0, 0.0, 0.5, 1.0]), chunk=chunk)


def _spec(case, seed):
    base = workloads.spec({2: "tiny", 3: "mid", 6: "heavy"}[case["classes"]])
    shape = dict(len_dist="pareto", max_len=16384, prompt_dist="lognormal", max_prompt=32768) if case["tail"] else \
        dict(len_dist="lognormal", max_len=4096, prompt_dist="uniform", max_prompt=2048)
    return dataclasses.replace(base, n_inst=case["inst"], n_active=case["held"], n_queued=case["queued"],
                               n_incoming=case["incoming"], slo_scale=case["slo"], drift_sigma=0.5,
                               occupancy_jitter=case["ragged"], seed=seed, **shape)


def prepare(case, seed):
    fl = workloads.make_fleet(_spec(case, seed))
    # (outputs are sized for full instances: how many requests uneven ones hold differs from seed to seed)
    M, R, na, nq = fl.n_inst, len(fl.in_prompt), case["inst"] * case["held"], len(fl.q_prompt)
    dev = torch.device("cuda", torch.cuda.current_device())

    def up(x):
        return torch.from_numpy(np.ascontiguousarray(x)).to(dev)

    d = {k: up(getattr(fl, k)) for k in ("act_off", "act_prompt", "act_gen", "act_rem", "act_rem_refreshed", "act_budget",
                                         "q_off", "q_prompt", "q_len", "in_prompt", "in_len", "in_budget")}
    # room for what feedback routing adds to an instance
    room = min(2048 - case["held"] - case["queued"], R) if case["call"] == "feedback" else 0
    h = binding.Fleet(fl.coef["delta"], fl.coef["alpha"], fl.coef["beta"], fl.coef["gamma"], fl.inst_class,
                      case["held"] + case["queued"] + room, int(fl.spec.max_len), max(R, 1))
    if case["blend"] > 0:
        for w, wait, prefill, decode in workloads.observed_status(fl, rounds=3, seed=seed):
            h.gr_observe(w, up(wait), up(prefill), up(decode))
        h.gr_set_blend(case["blend"])
    if case["caps"]:
        h.gr_set_batch_cap(workloads.batch_caps(fl, seed=seed))
    s = {"call": case["call"], "chunk": case["chunk"], "h": h, "d": d, "exclude": None}

    def out(n, dtype):
        return torch.zeros(n, dtype=dtype, device=dev)

    s["finish"], s["q_finish"] = out(na, torch.float32), out(nq, torch.float32)
    s["d_g"], s["rank"] = out(M, torch.float64), out(M, torch.int32)
    s["inst"], s["slack"], s["fallback"] = out(R, torch.int32), out(R, torch.float32), out(R, torch.uint8)
    if case["call"] in ("scan", "step"):
        s["flag"], s["new_finish"] = out(na, torch.uint8), out(na, torch.float32)
        s["target"], s["target_slack"], s["n_flagged"] = out(na, torch.int32), out(na, torch.float32), out(1, torch.int32)
    rng = np.random.Generator(np.random.PCG64([seed, 1]))
    if case["exclude"]:
        s["exclude"] = up(np.where(rng.random(R) < 0.5, rng.integers(0, M, R), -1).astype(np.int32))
    if case["call"] == "cached":
        s["hits"] = [up(x) for x in workloads.cached_prefixes(fl, 2.0, seed=seed)]
    if case["call"] == "route":
        _build(s)
    return s


def _build(s, everything=False):
    d = s["d"]
    if everything:
        s["h"].gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"],
                               d["q_len"], s["finish"], out_q_finish=s["q_finish"], out_d=s["d_g"], out_rank=s["rank"])
    else:
        s["h"].gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"],
                               d["q_len"], s["finish"])


def run(s):
    h, d, call = s["h"], s["d"], s["call"]
    routed = {"inst": s["inst"], "slack": s["slack"], "fallback": s["fallback"]}
    if call == "status":
        _build(s, everything=True)
        return {"finish": s["finish"], "q_finish": s["q_finish"], "d_g": s["d_g"], "rank": s["rank"]}
    got = {}
    if call in ("step", "refresh", "cached", "feedback"):
        _build(s)
        got["finish"] = s["finish"]
    if call in ("step", "refresh", "route"):
        h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], s["inst"], s["slack"], exclude_inst=s["exclude"],
                         out_fallback=s["fallback"])
        got.update(routed)
    elif call == "cached":
        h.gr_score_route_cached(d["in_prompt"], d["in_len"], d["in_budget"], *s["hits"], s["inst"], s["slack"],
                                exclude_inst=s["exclude"], out_fallback=s["fallback"])
        got.update(routed)
    elif call == "feedback":
        h.gr_route_feedback(s["chunk"], d["in_prompt"], d["in_len"], d["in_budget"], s["inst"], s["slack"],
                            exclude_inst=s["exclude"], out_fallback=s["fallback"])
        got.update(routed)
    if call in ("step", "scan"):
        h.gr_risk_scan(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem_refreshed"], d["q_off"], d["q_prompt"],
                       d["q_len"], d["act_budget"], s["flag"], s["new_finish"], s["target"], s["target_slack"],
                       s["n_flagged"])
        got.update(flag=s["flag"], new_finish=s["new_finish"], target=s["target"], target_slack=s["target_slack"],
                   n_flagged=s["n_flagged"])
    return got


def work(case):
    """Inputs read once and outputs written once; operations: the finish estimate of every held
    request (three running sums and one closed form, about 20 operations) once per status build.
    The selection's own operations depend on how the least latency is found and are left out."""
    M, R = case["inst"], case["incoming"]
    held = M * case["held"] * (0.625 if case["ragged"] else 1.0)
    queued = M * case["queued"]
    builds = {"route": 0, "step": 2}.get(case["call"], 1)
    by = builds * (held * 16 + queued * 8 + M * 8)          # prompt, generated, remaining; finish; offsets
    if case["call"] == "status":
        by += queued * 4 + M * 12                           # queued finish times, d_g, rank
    if case["call"] in ("step", "scan"):
        by += held * 13                                     # budget; flag, target, slack
    if R:
        by += R * (12 + 9 + (4 if case["exclude"] else 0))  # tokens, length, deadline; instance, slack, fallback
    if case["call"] == "cached":
        by += R * (4 + 2 * 8)
    return {"bytes": float(by), "flops": float(builds * (held + queued) * 20)}


def tolerance(case):
    """Times are single precision: a finish time is one rounding of a double, a latency four or five.
    Against the reference in double precision over the listed cases: relative 1.4e-7 in norm, 6.2e-6 at
    the worst value (slacks are differences), no decision different (2 of 10 million over all variants:
    two latencies, or a latency and a deadline, closer than a rounding).  Four times that is allowed."""
    return {"rel": 6e-7, "max": 2.5e-5, "differ": 1e-6}
