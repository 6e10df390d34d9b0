"""The native marshalling refuses what the binding's own check refuses, with the same errors; what only that
check can tell to be right (a subclass) passes.  Without it the same calls go by ctypes."""
import pytest
import torch

from paper_2605_16867_amd import binding


def _route(*tensors, handle=None):
    ctx0, length, budget, inst, slack = tensors
    return binding.marshal().score_route(handle, 4, ctx0, length, budget, None, inst, slack, None, None)


def test_refusals():
    cpu = torch.zeros(4, dtype=torch.int32)
    with pytest.raises(TypeError, match="ctx0: need a contiguous torch.int32 GPU tensor, got torch.int32 on cpu"):
        _route(cpu, cpu, cpu, cpu, cpu)
    with pytest.raises(AttributeError, match="numel"):
        _route([1], cpu, cpu, cpu, cpu)
    with pytest.raises(TypeError, match="arguments"):
        binding.marshal().score_route(None, 4)


@pytest.mark.gpu
def test_refusals_on_the_gpu():
    z = lambda n, t=torch.int32: torch.zeros(n, dtype=t, device="cuda:0")
    i, f = z(4), z(4, torch.float32)
    with pytest.raises(TypeError, match="budget: need a contiguous torch.float32 GPU tensor, got torch.int32"):
        _route(i, i, i, i, f)
    with pytest.raises(TypeError, match="pred_len: need a contiguous"):
        _route(i, z(8)[::2], f, i, f)
    with pytest.raises(ValueError, match="out_slack: 3 elements, need 4"):
        _route(i, i, f, i, f[:3])
    assert _route(i, i, f, i, f) == -1                      # (no handle: the library's own refusal)

    class Tensor(torch.Tensor):
        pass
    assert _route(i.as_subclass(Tensor), i, f, i, f) == -1
    with pytest.raises(TypeError, match="got torch.int32 on cpu"):
        _route(i, i.cpu().as_subclass(Tensor), f, i, f)


@pytest.mark.gpu
def test_the_current_stream():
    """A call goes to torch's current stream: behind what is queued there, with nothing else to wait for."""
    h = binding.Fleet([1e-5], [0.01], [1e-4], [1e-8], [0], 8, 100, 8)
    i32 = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda:0")
    side = torch.cuda.Stream()
    off, one = i32(0, 2), i32(5, 6)
    fin = torch.zeros(2, dtype=torch.float32, device="cuda:0")
    rem = i32(1, 1)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        rem.fill_(7)
        h.gr_build_status(off, one, one, rem, i32(0, 0), one[:0], one[:0], fin)
    torch.cuda.synchronize()
    late = fin.clone()
    h.gr_build_status(off, one, one, rem, i32(0, 0), one[:0], one[:0], fin)
    torch.cuda.synchronize()
    assert torch.equal(late, fin) and float(fin[0]) > 0.06
    h.close()


def test_without_the_native_module(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_marshal", None)
    monkeypatch.setattr(binding, "MARSHAL_PATH", str(tmp_path / "nowhere.so"))
    with pytest.warns(RuntimeWarning, match="marshalled by ctypes: .*nowhere.so is not built"):
        assert binding.marshal() is binding._Ctypes
    cpu = torch.zeros(4, dtype=torch.int32)
    with pytest.raises(TypeError, match="ctx0: need a contiguous torch.int32 GPU tensor, got torch.int32 on cpu"):
        _route(cpu, cpu, cpu, cpu, cpu)
    with pytest.raises(AttributeError, match="numel"):
        _route([1], cpu, cpu, cpu, cpu)
    (tmp_path / "nowhere.so").write_bytes(b"of another torch")
    monkeypatch.setattr(binding, "_marshal", None)
    with pytest.warns(RuntimeWarning, match="marshalled by ctypes"):
        binding.marshal()


@pytest.mark.gpu
def test_every_call_by_ctypes():
    """Both ways of handing over the arguments of the six calls of a serving loop: the same outputs, bit for bit."""
    from paper_2605_16867_amd import workloads
    from tests.parity import make_handle, upload
    fl = workloads.make_fleet(workloads.spec("tiny"))
    d, hits = upload(fl), [torch.from_numpy(x).cuda() for x in workloads.cached_prefixes(fl, 2.0, seed=1)]
    M, R, na, nq = fl.n_inst, len(fl.in_prompt), len(fl.act_prompt), len(fl.q_prompt)
    lists = [d[k] for k in ("act_off", "act_prompt", "act_gen", "act_rem", "q_off", "q_prompt", "q_len")]
    again = lists[:3] + [d["act_rem_refreshed"]] + lists[4:]
    req = [d[k] for k in ("in_prompt", "in_len", "in_budget")]
    ex = torch.arange(R, dtype=torch.int32, device="cuda:0") % M
    z = lambda n, t=torch.float32: torch.full((n,), 9, dtype=t, device="cuda:0")
    i32, u8 = torch.int32, torch.uint8
    seen = []
    for way in (binding.marshal(), binding._Ctypes):
        h = make_handle(fl, max_entries=64 + 8 + R)
        h._m, got = way, []
        choices = lambda: got.extend([z(R, i32), z(R), z(R, u8)]) or got[-3:]
        got += [z(na), z(nq), z(M, torch.float64), z(M, i32)]
        h.gr_build_status(*lists, got[0], out_q_finish=got[1], out_d=got[2], out_rank=got[3])
        T = [z(R * M), z(R * M)]
        got += T
        a, b, c = choices()
        h.gr_score_route(*req, a, b, exclude_inst=ex, out_fallback=c, out_T=T[0])
        a, b, c = choices()
        h.gr_score_route_noalloc(*req, a, b, exclude_inst=ex, out_fallback=c)
        a, b, c = choices()
        h.gr_score_route_cached(*req, *hits, a, b, exclude_inst=ex, out_fallback=c, out_T=T[1])
        a, b, c = choices()
        h.gr_route_feedback(3, *req, a, b, exclude_inst=ex, out_fallback=c)
        got += [z(na, u8), z(na), z(na, i32), z(na), z(1, i32)]
        h.gr_risk_scan(*again, d["act_budget"], *got[-5:])
        h.close()
        with pytest.raises(binding.GoodRouteError):
            h.gr_score_route(*req, a, b)
        seen.append(got)
    for a, b in zip(*seen):
        assert torch.equal(a, b)
