"""A risk scan whose running entries are not all in some instance's slice (offsets that begin late or end
early, instances that hold more than the handle was made for, entries without a token left under caps):
their flags are the caller's own, nobody sets them, and a request whose flag reads nonzero is scored like
any other flagged one.  Every target and slack against the pair-by-pair pass on the same request."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("caps", [False, True])
@pytest.mark.parametrize("n_inst,held", [(40, 20), (1100, 3), (560, 250)])
def test_flags_that_no_instance_sets(n_inst, held, caps):
    import torch
    rng = np.random.default_rng([n_inst, held])
    acts = [rand_entries(rng, held) for _ in range(n_inst)]
    na = n_inst * held
    allact = np.concatenate(acts)
    fl = fleet(rng.integers(0, 3, n_inst), acts, [[(500, 20)]] * n_inst, np.zeros((4096, 2)) + 1, np.ones(4096),
               act_budget=rng.uniform(0.5, 8, na) * solo(allact[:, 0] + allact[:, 1], allact[:, 2]))
    d = parity.upload(fl, "cuda:0")
    h = parity.make_handle(fl, max_entries=held + 1, max_requests=4096)
    if caps:
        h.gr_set_batch_cap(rng.integers(1, held + 3, n_inst))
    z = lambda n, t, v=0: torch.full((n,), v, dtype=t, device="cuda:0")
    flag, fin, tgt, tsl, nfl = z(na, torch.uint8), z(na, torch.float32), z(na, torch.int32, -7), z(na, torch.float32), z(1, torch.int32)

    def scan(off, rem):
        h.gr_risk_scan(off, d["act_prompt"], d["act_gen"], rem, d["q_off"], d["q_prompt"], d["q_len"], d["act_budget"],
                       flag, fin, tgt, tsl, nfl)
        torch.cuda.synchronize()

    scan(d["act_off"], d["act_rem"])         # in contract: every entry's instance is known from here on
    where = np.repeat(np.arange(n_inst), held)
    # the first and the last seventh in nobody's slice, one instance with three times its room
    off = np.clip(fl.act_off.astype(np.int64), na // 7, na - na // 7)
    g = n_inst // 2
    off[g:g + 3] = off[g]
    rem = fl.act_rem_refreshed.copy()
    if caps:
        rem[rng.random(na) < 0.1] = 0
    # lengths that only requests outside every slice have
    rem[: na // 7 : 3] = 4090 - np.arange(len(rem[: na // 7 : 3])) % 7
    flag.copy_(torch.from_numpy((rng.random(na) < 0.5).astype(np.uint8) * 3))
    scan(torch.from_numpy(off.astype(np.int32)).cuda(), torch.from_numpy(rem).cuda())
    for i in range(n_inst):
        where[off[i]:min(off[i + 1], off[i] + held + 1)] = i
    F, T, S = flag.cpu().numpy() != 0, tgt.cpu().numpy(), tsl.cpu().numpy()
    assert F[: na // 7].any() and F[-(na // 7):].any() and int(nfl.item()) == F.sum()
    assert np.all(T[~F] == -1) and np.all(S[~F] == 0)
    late = np.flatnonzero(F)
    for k in range(0, len(late), 4096):
        i = late[k:k + 4096]
        up = lambda x, t: torch.from_numpy(np.ascontiguousarray(x, dtype=t)).cuda()
        inst, slack = z(len(i), torch.int32, -7), z(len(i), torch.float32)
        h.gr_score_route_noalloc(up(fl.act_prompt[i] + fl.act_gen[i], np.int32), up(rem[i], np.int32), up(fl.act_budget[i], np.float32),
                                 inst, slack, exclude_inst=up(where[i], np.int32))
        torch.cuda.synchronize()
        assert np.array_equal(T[i], inst.cpu().numpy()) and np.array_equal(S[i], slack.cpu().numpy())
    h.close()


@pytest.mark.parametrize("case", ["no room", "no token"])
@pytest.mark.parametrize("n_inst,held,pairs", [(250, 250, None), (500, 70, None), (40, 20, None), (40, 20, 0), (600, 100, None)])
def test_offsets_that_cover_every_entry(n_inst, held, pairs, case):
    """The build alone says that there are entries whose flag it has not set: one instance holds more than the handle
    has room for, or, under caps, running entries have no token left.  Counted by the workgroups of a table that has
    a row for every length (250, 500, 40 instances), pair by pair (40), with the list of lengths (600: a class of 200)."""
    import torch
    rng = np.random.default_rng([n_inst, held, 1])
    acts = [rand_entries(rng, held * (2 if case == "no room" and g == n_inst // 3 else 1)) for g in range(n_inst)]
    all_ = np.concatenate(acts)
    na = len(all_)
    fl = fleet(np.arange(n_inst) % 3, acts, [[]] * n_inst, np.ones((8192, 2)), np.ones(8192),
               act_budget=rng.uniform(0.5, 8, na) * solo(all_[:, 0] + all_[:, 1], all_[:, 2]))
    d = parity.upload(fl, "cuda:0")
    h = parity.make_handle(fl, max_entries=held + 1, max_requests=8192)
    if pairs is not None:
        h.gr_set_small_batch_pairs(pairs)
    rem = fl.act_rem_refreshed.copy()
    if case == "no token":
        h.gr_set_batch_cap(rng.integers(1, held + 3, n_inst))
        rem[rng.random(na) < 0.1] = 0
    z = lambda n, t, v=0: torch.full((n,), v, dtype=t, device="cuda:0")
    fin, tgt, tsl, nfl = z(na, torch.float32), z(na, torch.int32, -7), z(na, torch.float32, 7), z(1, torch.int32, -7)
    first = torch.from_numpy((rng.random(na) < 0.5).astype(np.uint8) * 3).cuda()
    unset = np.zeros(na, bool)
    if case == "no room":
        a0 = fl.act_off[n_inst // 3]
        unset[a0 + held + 1:a0 + 2 * held] = True
    else:
        unset = rem == 0
    for _ in range(2):
        flag = first.clone()
        h.gr_risk_scan(d["act_off"], d["act_prompt"], d["act_gen"], torch.from_numpy(rem).cuda(), d["q_off"], d["q_prompt"],
                       d["q_len"], d["act_budget"], flag, fin, tgt, tsl, nfl)
        torch.cuda.synchronize()
        assert (flag.cpu().numpy()[unset] == 3).any()       # (the library sets 0 or 1)
        off = flag == 0
        assert int(nfl.item()) == int((~off).sum())
        assert bool((tgt[off] == -1).all()) and bool((tsl[off] == 0).all())
    h.close()
