"""The table of long-tailed fleets, where an instance has no, a few or many entries in a block of lengths: every pair's
latency against the pair-by-pair pass, bit for bit, with lengths on and next to the instances' own."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu


MAX_LEN = 16384


@pytest.mark.parametrize("cap", [64, 256, 512, 1024])
@pytest.mark.parametrize("spread", ["short", "far", "crowded"])
def test_every_latency(cap, spread):
    """short: nearly all entries in the first blocks; far: one in a block here and there; crowded: 15 to 17 and 63 to 65
    neighbours in the middle of a block, between blocks that hold none.  Two classes are too large for a row per length, and
    the batch too small for the classes to be looked at first: the ordinary table (tables of up to 512 lengths are read whole)."""
    import torch
    dev = "cuda:0"
    rng = np.random.default_rng(cap)
    acts = []
    for g in range(290):
        n = int(rng.choice([0, 1, cap // 2, cap - 1, cap]))
        e = rand_entries(rng, n)
        if spread == "short":
            e[:, 2] = np.minimum(1 + (30 * (rng.random(n) ** -0.8 - 1)).astype(np.int64), MAX_LEN)
        elif spread == "far":
            e[:, 2] = rng.integers(1, MAX_LEN + 1, n)
        else:
            k = int(rng.choice([1, 4, 15, 16, 17, 63, 64, 65]))
            e[:, 2] = np.where(np.arange(n) < k, 6000 + rng.integers(0, 40, n), np.where(np.arange(n) % 2, 3, 16000))
        acts.append(e)
    lens = np.concatenate([np.arange(1, MAX_LEN + 1), rng.integers(1, MAX_LEN + 1, 100)])      # (a row for each, and on the entries' own)
    rng.shuffle(lens)
    inc = np.stack([rng.integers(128, 2049, len(lens)), lens], 1)
    fl = fleet(np.arange(290) % 2, acts, [[]] * 290, inc, 3.0 * solo(inc[:, 0], inc[:, 1]), max_len=MAX_LEN)
    d = parity.upload(fl, dev)
    h = parity.make_handle(fl, max_entries=cap)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device=dev)
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)

    def routed(at, n):
        out = [torch.full((n,), -7, dtype=torch.int32, device=dev), torch.zeros(n, dtype=torch.float32, device=dev),
               torch.zeros(n, 290, dtype=torch.float32, device=dev)]
        h.gr_score_route(*(d[k][at:at + n] for k in ("in_prompt", "in_len", "in_budget")), out[0], out[1], out_T=out[2])
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in out]

    h.gr_set_small_batch_pairs(0)
    table = routed(0, len(lens))
    h.gr_set_small_batch_pairs(1 << 40)
    for at in range(0, len(lens), 4096):
        n = min(4096, len(lens) - at)
        for a, b in zip(table, routed(at, n)):
            assert np.array_equal(a[at:at + n], b)
    assert h.gr_device_status() == 0
    h.close()


PER_CLASS = 516      # two classes of 33 runs of 16; whole groups of four, which a wave of the table takes


def _crowds(rng, spread, cap):
    """The remaining lengths of an instance each, as many for all of them, so that contexts alone order a class."""
    if spread in ("short", "far"):
        n = cap - cap // 8
        for _ in range(2 * PER_CLASS):
            yield np.minimum(1 + (30 * (rng.random(n) ** -0.8 - 1)).astype(np.int64), MAX_LEN) if spread == "short" else \
                rng.integers(1, MAX_LEN + 1, n)
        return
    # four neighbours in the order together have `total` entries in block 23 of 256 lengths, behind 0 to 15 that are shorter
    n, first = min(cap, 100), 23 * 256 + 1
    for group in range(2 * PER_CLASS // 4):
        total = [0, 1, 15, 16, 17, 18, 24, 40, 100, 250][group % 10]
        share = rng.multinomial(total, [0.25] * 4 if group % 3 else [1, 0, 0, 0])
        for k in np.minimum(share, n - 16):
            inside = first + rng.choice([0, 1, 3, 4, 100, 128, 254, 255], k) if group % 2 else first + rng.integers(0, 256, k)
            before = rng.integers(1, first, rng.integers(0, 16))
            yield np.concatenate([before, inside, rng.choice([first + 256, 16000, MAX_LEN], n - k - len(before))])


@pytest.mark.parametrize("cap", [64, 256, 512])
@pytest.mark.parametrize("spread", ["short", "far", "counted"])
@pytest.mark.parametrize("gaps", [False, True])
def test_every_latency_classes_first(cap, spread, gaps):
    """Batches and fleets large enough for the classes to be looked at first, with tables of no more than eight lengths to a
    block of rows: waves whose instances have few entries in a block go through those.  counted: a wave's four
    instances have 15 to 17 and other numbers of them together, on a block's first and last rows among others.
    gaps: entries of lengths that have no row, and a last block that is not full."""
    import torch
    dev = "cuda:0"
    rng = np.random.default_rng([cap, gaps])
    acts = [np.stack([np.full(len(R), 100 + g % PER_CLASS), np.zeros(len(R), np.int64), R], 1) for g, R in enumerate(_crowds(rng, spread, cap))]
    lens = np.arange(1, MAX_LEN + 1)
    if gaps:
        lens = lens[(rng.random(MAX_LEN) < 0.9) & (lens < 16100)]
    rng.shuffle(lens)
    n, M = len(lens), 2 * PER_CLASS
    inc = np.stack([rng.integers(128, 2049, n), lens], 1)
    fl = fleet(np.arange(M) // PER_CLASS, acts, [[]] * M, inc, 3.0 * solo(inc[:, 0], inc[:, 1]), max_len=MAX_LEN)
    d = parity.upload(fl, dev)
    times = -(-(1 << 17) // n)
    h = parity.make_handle(fl, max_entries=cap, max_requests=n * times)
    fin = torch.zeros(len(fl.act_prompt), dtype=torch.float32, device=dev)
    h.gr_build_status(d["act_off"], d["act_prompt"], d["act_gen"], d["act_rem"], d["q_off"], d["q_prompt"], d["q_len"], fin)

    def routed(*req):
        n = len(req[0])
        out = [torch.full((n,), -7, dtype=torch.int32, device=dev), torch.zeros(n, dtype=torch.float32, device=dev),
               torch.zeros(n, M, dtype=torch.float32, device=dev)]
        h.gr_score_route(*req, out[0], out[1], out_T=out[2])
        return out

    req = [d[k] for k in ("in_prompt", "in_len", "in_budget")]
    h.gr_set_small_batch_pairs(0)
    h.gr_profile_enable(32)
    table = routed(*(x.repeat(times) for x in req))
    assert h.gr_profile_read()["k_class<route>"][1] == 1
    h.gr_profile_enable(0)
    h.gr_set_small_batch_pairs(1 << 40)
    for at in range(0, n, 4096):
        want = routed(*(x[at:at + 4096] for x in req))
        for a, b in zip(table, want):
            assert all(torch.equal(a[t * n + at:t * n + at + len(b)], b) for t in range(times))
    assert h.gr_device_status() == 0
    h.close()
