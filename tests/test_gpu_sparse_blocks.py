"""The table of long-tailed fleets, where an instance has no, a few or many entries in a block of lengths: every pair's
latency against the pair-by-pair pass, bit for bit, with lengths on and next to the instances' own."""
import numpy as np
import pytest

from tests import parity
from tests.fleets import fleet, rand_entries, solo

pytestmark = pytest.mark.gpu


MAX_LEN = 16384


@pytest.mark.parametrize("cap", [64, 256, 512, 1024])      # (tables of up to 512 are taken that way)
@pytest.mark.parametrize("spread", ["short", "far", "crowded"])
def test_every_latency(cap, spread):
    """short: nearly all entries in the first blocks; far: one in a block here and there; crowded: 15 to 17 and 63 to 65
    neighbours in the middle of a block, between blocks that hold none.  Two classes are too large for a row per length."""
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
