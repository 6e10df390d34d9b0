"""Feedback routing whose rounds are one launch, against the same rounds through the table of lengths and a rebuild each, bit for bit: by all
workgroups together, by a part of them and by one alone (those that have come in time, or as many as the caller allows),
lists of several blocks, several fleets at once on a stream each, and recorded and replayed.  Where its workgroups do not fit the
compute units, each round is a launch."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2605_16867_amd import binding, workloads
from tests.parity import upload

pytestmark = pytest.mark.gpu


def _fleet(n_inst, held, n, slo, seed):
    return workloads.make_fleet(dataclasses.replace(workloads.spec("mid"), n_inst=n_inst, n_active=held, n_queued=held // 10,
                                                    n_incoming=n, slo_scale=slo, occupancy_jitter=True, seed=seed))


class _Routing:
    def __init__(self, fl, chunk, entries, pairs=None, looks=None, blend=0.0, team=None):
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
        self.chunk, self.n, self.d = chunk, len(fl.in_prompt), upload(fl)
        self.h = binding.Fleet(fl.coef["delta"], fl.coef["alpha"], fl.coef["beta"], fl.coef["gamma"], fl.inst_class, entries,
                               int(fl.spec.max_len), self.n)
        if pairs is not None:
            self.h.gr_set_small_batch_pairs(pairs)
        if looks is not None:
            self.h.gr_set_feedback_wait(looks)
        if team is not None:
            self.h.gr_set_feedback_team(team)
        if blend:
            for w, wait, prefill, decode in workloads.observed_status(fl, rounds=2, seed=3):
                self.h.gr_observe(w, dev(wait), dev(prefill), dev(decode))
            self.h.gr_set_blend(blend)
        z = lambda t, v=0: torch.full((self.n,), v, dtype=t, device="cuda")
        self.fin = torch.zeros(max(len(fl.act_prompt), 1), device="cuda")
        self.exclude = dev(np.where(np.arange(self.n) % 3 == 0, np.arange(self.n) % fl.n_inst, -1).astype(np.int32))
        self.out = [z(torch.int32, -7), z(torch.float32), z(torch.uint8, 9)]
        self.after = [z(torch.int32, -7), z(torch.float32), z(torch.uint8, 9)]

    def run(self):
        d = self.d
        self.h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], self.fin)
        self.h.gr_route_feedback(self.chunk, d["in_prompt"], d["in_len"], d["in_budget"], self.out[0], self.out[1],
                                 exclude_inst=self.exclude, out_fallback=self.out[2])
        self.h.gr_score_route(d["in_prompt"], d["in_len"], d["in_budget"], self.after[0], self.after[1], out_fallback=self.after[2])

    def result(self):
        torch.cuda.synchronize()
        assert self.h.gr_device_status() == 0
        return [x.clone() for x in self.out + self.after]


@pytest.mark.parametrize("n_inst,held,entries,chunk,n,slo", [
    (1, 5, 700, 4, 600, 16.0), (3, 20, 500, 1, 160, 1.0), (5, 30, 1024, 4, 400, 16.0), (17, 10, 128, 3, 90, 4.0), (64, 200, 512, 8, 300, 16.0),
    (256, 100, 2048, 64, 700, 16.0), (257, 60, 400, 30, 300, 1.0), (400, 30, 300, 3, 60, 16.0), (512, 40, 256, 64, 450, 4.0)])
@pytest.mark.parametrize("blend", [0.0, 0.5])
def test_together_and_alone(n_inst, held, entries, chunk, n, slo, blend):
    fl = _fleet(n_inst, held, n, slo, n_inst + chunk)
    got = []
    groups = (n_inst + 3) // 4
    for pairs, looks, team in ((0, None, None), (None, None, None), (None, 0, None), *((None, None, k) for k in {1, groups // 3, groups - 1} if k > 0)):
        r = _Routing(fl, chunk, entries, pairs, looks, blend, team)
        r.run()
        got.append(r.result())
        shared = r.h.gr_feedback_team()
        assert shared == (0 if pairs == 0 else team or groups) if looks is None else 1 <= shared <= groups
        r.h.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)


# Sizes on either side of the choice: rounds in all, instances, and requests of a chunk that the gain of a round is weighed against.
@pytest.mark.parametrize("n_inst,chunk,n,one", [
    (512, 1, 2, False), (64, 1, 3, False), (65, 1, 3, True), (128, 19, 57, True), (128, 20, 60, False), (4, 15, 60, True), (4, 16, 64, False),
    (4, 16, 65, True), (1, 16, 64, False), (1, 14, 56, True), (64, 44, 924, True), (64, 46, 966, False), (256, 64, 193, True), (256, 63, 189, False)])
def test_where_rounds_are_one_launch(n_inst, chunk, n, one):
    fl = _fleet(n_inst, 70, n, 4.0, n_inst + n)
    got = []
    for pairs in (0, None):
        r = _Routing(fl, chunk, 700, pairs)
        r.run()
        got.append(r.result())
        assert r.h.gr_feedback_team() == ((n_inst + 3) // 4 if one and pairs is None else 0)
        r.h.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)


# (four of 512 instances do not fit side by side: each gets a part of the chip, and goes on with the workgroups that have started)
@pytest.mark.parametrize("fleets,looks", [(((256, 32), (300, 24)), None), (((512, 16),) * 4, None), (((512, 16),) * 4, 2)])
def test_several_at_once(fleets, looks):
    rs, wants = [], []
    for k, (n_inst, chunk) in enumerate(fleets):
        fl = _fleet(n_inst, 80, 500, (1.0, 16.0)[k % 2], 40 + k)
        want = _Routing(fl, chunk, 600, pairs=0)
        want.run()
        wants.append(want.result())
        rs.append(_Routing(fl, chunk, 600, looks=looks))
    streams = [torch.cuda.Stream() for _ in rs]
    torch.cuda.synchronize()
    for _ in range(4):
        for r, s in zip(rs, streams):
            with torch.cuda.stream(s):
                r.run()
    for r, want in zip(rs, wants):
        for a, b in zip(r.result(), want):
            assert torch.equal(a, b)


def test_recorded():
    fl = _fleet(256, 90, 400, 4.0, 9)
    want = _Routing(fl, 16, 700, pairs=0)
    want.run()
    expected = want.result()
    r = _Routing(fl, 16, 700)
    r.run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        r.run()
    for _ in range(4):
        for x in r.out + r.after:
            x.fill_(3)
        graph.replay()
        for a, b in zip(r.result(), expected):
            assert torch.equal(a, b)
        r.run()      # (a direct call between the replays)
        for a, b in zip(r.result(), expected):
            assert torch.equal(a, b)


# A workgroup for every four instances: on as many compute units as there are of those, and one fewer.
@pytest.mark.parametrize("n_inst", [5, 8, 254])
def test_a_launch_for_each_round_where_the_workgroups_do_not_fit(n_inst):
    fl = _fleet(n_inst, 60, 200, 4.0, n_inst)
    groups, rounds = (n_inst + 3) // 4, 25
    got, launches = [], []
    for units in (None, groups, groups - 1, 0):
        r = _Routing(fl, 8, 500)
        if units is not None:
            r.h.gr_set_feedback_units(units)
        r.h.gr_profile_enable(200)
        r.run()
        got.append(r.result())
        launches.append(r.h.gr_profile_read()["k_feedback"][1])
        r.h.close()
    assert launches[0] == launches[1] < 6
    assert launches[2] == launches[3] == rounds + 1
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)
