"""The stream an execute call is enqueued on: the given one, or torch's current one on the current device."""
import pytest

from paper_2609_34645_amd import emu


@pytest.mark.gpu
def test_calls_follow_the_current_stream(gpu_lib):
    import torch

    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    assert emu._stream_handle(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(a):
        assert emu._stream_handle(None) == a.cuda_stream
        assert emu._stream_handle(b) == b.cuda_stream
        with torch.cuda.stream(b):
            assert emu._stream_handle(None) == b.cuda_stream
        assert emu._stream_handle(None) == a.cuda_stream
    assert emu._stream_handle(None) == torch.cuda.current_stream().cuda_stream


@pytest.mark.gpu
def test_a_call_waits_for_its_streams_work(gpu_lib):
    """Source writes queued on a side stream before the call, on that stream, are what the call moves."""
    import torch

    m = emu.Model(1, 64, 2, 32, 2, 64, 4096)
    plan = emu.Plan(emu.Layout(m, 1, 1), emu.Layout(m, 2, 1))
    ws = plan.workspace()
    S, D = plan.alloc(0, fill=0), plan.alloc(1, fill=0)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        x = torch.randn(2048, 2048, device="cuda")
        for _ in range(20):
            x = x @ x * 1e-3  # work ahead of the write
        for buf in S.bufs:
            buf.fill_(7)
        plan.reshard(ws, S.ptrs, D.ptrs)
    side.synchronize()
    for t in D.tensors:
        assert bool((t == 7).all())
