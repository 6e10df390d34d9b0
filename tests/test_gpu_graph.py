"""The three calls recorded into a HIP graph and replayed.

A serving loop that routes batch after batch is bound by launch cost when the
batches are small; the calls only launch kernels on the caller's stream (no
allocation, no copy, no host synchronisation, no memset node), so they can be
captured once and replayed.  Every replay is checked against the same calls
made directly, on inputs that change between replays, with the program's own
direct work and synchronisations in between.
"""
import numpy as np
import pytest

from paper_2605_16867_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu

INPUTS = ("act_prompt", "act_gen", "act_rem", "act_rem_refreshed", "act_budget", "q_prompt", "q_len",
          "in_prompt", "in_len", "in_budget")


def _outputs(torch, na, R, dev):
    z = lambda n, t: torch.zeros(n, dtype=t, device=dev)
    return dict(fin=z(na, torch.float32), inst=z(R, torch.int32), slack=z(R, torch.float32),
                fb=z(R, torch.uint8), flag=z(na, torch.uint8), fin2=z(na, torch.float32),
                tgt=z(na, torch.int32), tsl=z(na, torch.float32), nfl=z(1, torch.int32))


def _three_calls(h, d, o):
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"],
                      d["q_off"], d["q_prompt"], d["q_len"], o["fin"])
    h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], o["inst"], o["slack"], out_fallback=o["fb"])
    h.gr_risk_scan(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem_refreshed"],
                   d["q_off"], d["q_prompt"], d["q_len"], d["act_budget"],
                   o["flag"], o["fin2"], o["tgt"], o["tsl"], o["nfl"])


@pytest.mark.parametrize("name,small_batch_pairs", [("mid", None), ("mid", 0), ("tiny", None), ("large", None)])
def test_replays_equal_direct_calls(name, small_batch_pairs):
    import torch
    dev = "cuda:0"
    # same shapes (offsets), different contents: seeds change lengths, prompts and budgets only
    fleets = [workloads.make_fleet(workloads.spec(name, seed=s, slo_scale=sc))
              for s, sc in ((0, 1.0), (1, 3.0), (2, 8.0), (3, 1.5))]
    for fl in fleets[1:]:
        assert np.array_equal(fl.act_off, fleets[0].act_off) and np.array_equal(fl.q_off, fleets[0].q_off)
        assert len(fl.in_prompt) == len(fleets[0].in_prompt)
    ups = [parity.upload(fl, dev) for fl in fleets]
    na, R = len(fleets[0].act_prompt), len(fleets[0].in_prompt)

    parity.SMALL_BATCH_PAIRS = small_batch_pairs
    try:
        h_graph, h_direct = parity.make_handle(fleets[0]), parity.make_handle(fleets[0])
    finally:
        parity.SMALL_BATCH_PAIRS = None
    d = {k: v.clone() for k, v in ups[0].items()}       # the buffers the graph reads
    o_graph, o_direct = _outputs(torch, na, R, dev), _outputs(torch, na, R, dev)

    # warm up on a side stream (first launches set kernel attributes), then record
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        _three_calls(h_graph, d, o_graph)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _three_calls(h_graph, d, o_graph)

    for rep, up in enumerate(ups[1:] + ups[:1]):
        for k in INPUTS:
            d[k].copy_(up[k])
        for v in o_graph.values():
            v.fill_(7)
        graph.replay()
        _three_calls(h_direct, up, o_direct)      # the same work made directly, on another handle
        torch.cuda.synchronize()
        for k in o_graph:
            a, b = o_graph[k].cpu().numpy(), o_direct[k].cpu().numpy()
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), f"replay {rep}: {k} differs from the direct call"
        assert int(o_graph["nfl"].item()) == int(o_graph["flag"].sum().item())
    h_graph.close()
    h_direct.close()


@pytest.mark.parametrize("entry,small_batch_pairs", [("gr_score_route", None), ("gr_score_route", 0),
                                                     ("gr_score_route_noalloc", None)])
def test_a_recorded_routing_call_follows_status_builds_made_outside_the_graph(entry, small_batch_pairs):
    """Only the routing call is recorded; the status is rebuilt by direct calls between replays.
    A recorded scoring pass makes the capability order of whatever status it finds."""
    import torch
    dev = "cuda:0"
    fleets = [workloads.make_fleet(workloads.spec("mid", seed=s, slo_scale=sc, n_incoming=1024))
              for s, sc in ((0, 2.0), (1, 3.0), (2, 8.0))]
    ups = [parity.upload(fl, dev) for fl in fleets]
    na, R = len(fleets[0].act_prompt), len(fleets[0].in_prompt)
    parity.SMALL_BATCH_PAIRS = small_batch_pairs
    try:
        h_graph, h_direct = parity.make_handle(fleets[0]), parity.make_handle(fleets[0])
    finally:
        parity.SMALL_BATCH_PAIRS = None
    d = {k: v.clone() for k, v in ups[0].items()}
    o_graph, o_direct = _outputs(torch, na, R, dev), _outputs(torch, na, R, dev)

    def build(h, src, o):
        h.gr_build_status(src["act_off"], src["act_prompt"], src["act_gen"], src["act_rem"],
                          src["q_off"], src["q_prompt"], src["q_len"], o["fin"])

    def route(h, src, o):
        getattr(h, entry)(src["in_prompt"], src["in_len"], src["in_budget"], o["inst"], o["slack"], out_fallback=o["fb"])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        build(h_graph, d, o_graph)
        route(h_graph, d, o_graph)            # the capability order of this status now exists
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        route(h_graph, d, o_graph)

    for rep, up in enumerate(ups[1:] + ups[:1]):
        for k in INPUTS:
            d[k].copy_(up[k])
        for k in ("inst", "slack", "fb"):
            o_graph[k].fill_(7)
        build(h_graph, d, o_graph)            # a direct call: another status, another capability order
        graph.replay()
        build(h_direct, up, o_direct)
        route(h_direct, up, o_direct)
        torch.cuda.synchronize()
        for k in ("fin", "inst", "slack", "fb"):
            a, b = o_graph[k].cpu().numpy(), o_direct[k].cpu().numpy()
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), f"replay {rep}: {k} differs from the direct call"
    assert len({tuple(workloads.make_fleet(workloads.spec("mid", seed=s)).act_rem[:8]) for s in (0, 1, 2)}) == 3
    h_graph.close()
    h_direct.close()


# ---- what a recording, and its replays, leave to the direct calls on the same handle
def _warm_stream(torch):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    return side


def _build(h, src, o):
    h.gr_build_status(src["act_off"], src["act_prompt"], src["act_gen"], src["act_rem"],
                      src["q_off"], src["q_prompt"], src["q_len"], o["fin"])


def _route(h, src, o):
    h.gr_score_route(src["in_prompt"], src["in_len"], src["in_budget"], o["inst"], o["slack"], out_fallback=o["fb"])


def _route_cached(h, src, o):
    import torch
    R = len(src["in_prompt"])
    off = torch.arange(R + 1, dtype=torch.int32, device="cuda:0")
    where = torch.arange(R, dtype=torch.int32, device="cuda:0") % h.n_inst
    h.gr_score_route_cached(src["in_prompt"], src["in_len"], src["in_budget"], off, where, src["in_prompt"] // 2,
                            o["inst"], o["slack"], out_fallback=o["fb"])


def _equal(torch, a, b, keys=("inst", "slack", "fb")):
    torch.cuda.synchronize()
    for k in keys:
        x, y = a[k].cpu().numpy(), b[k].cpu().numpy()
        assert np.array_equal(x, y, equal_nan=x.dtype.kind == "f"), f"{k}: {(x != y).sum()} of {len(x)} differ"


def _mid(n):
    fls = [workloads.make_fleet(workloads.spec("mid", seed=s, slo_scale=8.0, n_incoming=1024)) for s in range(n)]
    return fls, [parity.upload(fl, "cuda:0") for fl in fls]


@pytest.mark.parametrize("call", [_route, _route_cached])
@pytest.mark.parametrize("first_order", [True, False])
def test_a_direct_call_after_a_recording_that_was_not_replayed(call, first_order):
    """Recording a routing call runs nothing: the next direct call makes the class order itself, whether
    an earlier status had one or none was ever made."""
    import torch
    fls, ups = _mid(2)
    na, R = len(fls[0].act_prompt), len(fls[0].in_prompt)
    h, fresh = parity.make_handle(fls[0]), parity.make_handle(fls[0])
    for x in (h, fresh):
        x.gr_set_small_batch_pairs(0)
    o, want, rec = (_outputs(torch, na, R, "cuda:0") for _ in range(3))
    if first_order:
        _build(h, ups[0], o)
        call(h, ups[0], o)
    _build(h, ups[1], o)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _route(h, ups[1], rec)
    call(h, ups[1], o)
    _build(fresh, ups[1], want)
    call(fresh, ups[1], want)
    _equal(torch, o, want)
    graph.replay()
    _route(fresh, ups[1], want)
    _equal(torch, rec, want)
    h.close()
    fresh.close()


@pytest.mark.parametrize("call", [_route, _route_cached])
def test_a_direct_call_after_replays_of_a_recorded_build(call):
    """Only the status build is recorded: every replay is another status under the direct calls."""
    import torch
    fls, ups = _mid(3)
    na, R = len(fls[0].act_prompt), len(fls[0].in_prompt)
    h, fresh = parity.make_handle(fls[0]), parity.make_handle(fls[0])
    for x in (h, fresh):
        x.gr_set_small_batch_pairs(0)
    d = {k: v.clone() for k, v in ups[0].items()}
    o, want = (_outputs(torch, na, R, "cuda:0") for _ in range(2))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _build(h, d, o)
    # (before the first replay there is no status, whatever the recording: any answer is fine as long
    # as it names instances)
    call(h, d, o)
    torch.cuda.synchronize()
    assert bool(((o["inst"] >= -1) & (o["inst"] < h.n_inst)).all())
    for up in ups[1:] + ups[:1]:
        for k in INPUTS:
            d[k].copy_(up[k])
        graph.replay()
        call(h, up, o)
        _build(fresh, up, want)
        call(fresh, up, want)
        _equal(torch, o, want)
    h.close()
    fresh.close()


def test_a_recorded_build_of_another_blend_weight():
    """The classes decide a large batch by themselves only where no status has a blend: not to be taken from
    the weight of a build that has only been recorded, nor from that of the last direct one when
    a replay has put another status in its place."""
    import torch
    from tests.test_gpu_runs import _fleet
    fl = _fleet(1300, 3, (1 << 17) + 3, "mixed")
    d = parity.upload(fl, "cuda:0")
    na, R, M = len(fl.act_prompt), len(fl.in_prompt), 1300
    h, fresh = parity.make_handle(fl), parity.make_handle(fl)
    rng = np.random.default_rng(1)
    obs = [torch.from_numpy(rng.uniform(lo, hi, M).astype(np.float32)).cuda() for lo, hi in
           ((0.0, 20.0), (1e-5, 2e-4), (0.02, 0.4))]
    for x in (h, fresh):
        x.gr_observe(1.0, *obs)
    o, want = (_outputs(torch, na, R, "cuda:0") for _ in range(2))

    def expect(weight):
        fresh.gr_set_blend(weight)
        _build(fresh, d, want)
        _route(fresh, d, want)
        _route(h, d, o)
        _equal(torch, o, want)

    for direct, recorded in ((0.5, 0.0), (0.0, 0.5)):
        h.gr_set_blend(direct)
        _build(h, d, o)
        h.gr_set_blend(recorded)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _build(h, d, o)
        expect(direct)          # not replayed: the direct build's status
        graph.replay()
        expect(recorded)
    h.close()
    fresh.close()


@pytest.mark.parametrize("replayed", [False, True])
def test_feedback_after_a_recorded_build(replayed):
    """The first rebuild of a feedback call takes every instance when the tables are not known to be of
    the weight in force: a build that was only recorded has not made them so, and a replay
    of one may have brought back tables of another weight."""
    import torch
    fls, ups = _mid(1)
    fl, d = fls[0], ups[0]
    na, R, M = len(fl.act_prompt), len(fl.in_prompt), fl.n_inst
    h, fresh = (parity.make_handle(fl, max_entries=1024) for _ in range(2))
    rng = np.random.default_rng(2)
    obs = [torch.from_numpy(rng.uniform(lo, hi, M).astype(np.float32)).cuda() for lo, hi in
           ((0.0, 20.0), (1e-5, 2e-4), (0.02, 0.4))]
    o, want = (_outputs(torch, na, R, "cuda:0") for _ in range(2))
    for x, out in ((h, o), (fresh, want)):
        x.gr_observe(1.0, *obs)
        if not replayed:
            _build(x, d, out)
            x.gr_set_blend(0.5)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _build(h, d, o)         # weight 0.5 if it is never replayed, else 0
    if replayed:
        h.gr_set_blend(0.5)
        _build(h, d, o)
        graph.replay()          # tables of weight 0 again
        _build(fresh, d, want)
        fresh.gr_set_blend(0.5)

    def feedback(x, out):
        n = 6                   # few requests: most instances are given nothing
        x.gr_route_feedback(2, d["in_prompt"][:n], d["in_len"][:n], d["in_budget"][:n], out["inst"][:n], out["slack"][:n])
        _route(x, d, out)

    feedback(h, o)
    feedback(fresh, want)
    _equal(torch, o, want)
    h.close()
    fresh.close()
