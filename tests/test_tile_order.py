"""The order in which workgroups take tiles: every tile is moved once, whatever the map's length."""
import pytest

from paper_2609_34645_amd import emu


@pytest.mark.gpu
@pytest.mark.parametrize("vocab", [31 * 1024, 32 * 1024 - 40, 32 * 1024, 32 * 1024 + 33, 65 * 1024 + 7, 3 * 32 * 1024 - 64,
                                   4 * 32 * 1024 - 1000, 4 * 32 * 1024, 5 * 32 * 1024 + 33])
@pytest.mark.parametrize("pad", [0, 96])
def test_maps_around_whole_rounds_of_blocks(gpu_lib, vocab, pad):
    """Maps of about one to five rounds of 8 x 256 tiles of 4 KB, a few tiles short of one and past it, and on both
    sides of the four rounds from which the order goes by blocks, with and without a zero-fill section behind the
    copies; streaming, and written through."""
    import torch
    from test_any_alignment import run_through

    m = emu.Model(1, 64, 2, 32, 2, 64, vocab)
    plan = emu.Plan(emu.Layout(m, 1, 1), emu.Layout(m, 1, 1, pad))
    ws = plan.workspace()
    S, D = plan.alloc(0, guard=256), plan.alloc(1, fill=0xA5, guard=256)
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab)
    for b in S.bufs:
        b.copy_(torch.randint(0, 256, b.shape, generator=g, device="cuda", dtype=torch.uint8))
    plan.reshard(ws, S.ptrs, D.ptrs)
    torch.cuda.synchronize()
    assert plan.info["n_zero_segments"] == (2 if pad and vocab % pad else 0)
    for s, d in zip(S.tensors, D.tensors):
        assert torch.equal(d[:s.numel()], s)
        assert not bool(d[s.numel():].any())
    run_through(plan, ws, S, D)
