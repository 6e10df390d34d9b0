"""The native marshalling refuses what the binding's own check refuses, with the same errors; what only that
check can tell to be right (a subclass) passes."""
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
