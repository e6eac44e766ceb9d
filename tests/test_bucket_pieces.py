"""Pack and unpack of pieces at every length and phase: against each rank's stream, put together by torch."""
import pytest

from paper_2609_34645_amd import emu

# Bucket sizes: a few elements; around one and two units of 16 bytes; around a 4 KB chunk, with odd sizes that
# put bucket k at any phase; larger than any stream (the division by the bucket size at its extremes)
SIZES = [4, 12, 16, 20, 28, 44, 4092, 4096, 4100, 6140, 12292, (1 << 33) + 4, 1 << 63]


# Sets large enough to write through at these bucket sizes, as (shape, vocabulary padding, element type, sizes):
# tensors off the 4 KB grid (odd widths) and on it, buckets on it and off it, at phases 0, 2, 4, 8 and 12 of a vector
LARGE = [((4, 996, 12, 83, 6, 2658, 50257), 64, "bf16", [1 << 22, (1 << 22) + 2, (1 << 20) - 4, (1 << 24) + 8, (1 << 16) + 14]),
         ((4, 996, 12, 83, 6, 2658, 50257), 64, "fp32", [1 << 22, (1 << 22) + 4, (1 << 24) - 8]),
         ((1, 2048, 32, 64, 8, 5632, 32000), 0, "bf16", [1 << 26, (1 << 26) - 2, (1 << 22) + 16])]


def check(lay, sizes):
    """Pack and unpack at every size: each bucket is its part of the rank's stream, and the tensors come back."""
    import torch
    from gpu_util import Guard

    plan = emu.Plan(lay, lay)
    ws = plan.workspace()
    S = plan.alloc(0, guard=64)
    g = torch.Generator(device="cuda")
    g.manual_seed(lay.model.hidden)
    for b in S.bufs:
        b.copy_(torch.randint(0, 256, b.shape, generator=g, device="cuda", dtype=torch.uint8))
    ranks = {}
    for d, t in zip(plan.tensors(0), S.tensors):
        ranks.setdefault(d["rank"], []).append(t)
    streams = {r: torch.cat(ts) for r, ts in ranks.items()}
    for B in sizes:
        bufs, bptrs = plan.alloc_buckets(0, B, fill=0xA5, guard=64)
        R = plan.alloc(0, fill=0x5A, guard=64)
        guard = Guard(keep=S.tensors, fills=[(bufs, 0xA5), (R.tensors, 0x5A)], snapshot="device", label=f"B={B}")
        plan.pack(ws, 0, B, S.ptrs, bptrs)
        plan.unpack(ws, 0, B, bptrs, R.ptrs)
        torch.cuda.synchronize()
        guard.check()
        for i, b in zip(plan.bucket_info(0, B), bufs):
            want = streams[i["rank"]][i["stream_offset"]:i["stream_offset"] + i["bytes"]]
            assert torch.equal(b, want), (B, i)
        for i, (s, r) in enumerate(zip(S.tensors, R.tensors)):
            assert torch.equal(s, r), (B, i)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("tiles", [1, 0], ids=["tile_per_wg", "persistent"])
def test_pieces(gpu_lib, dtype, tiles):
    old = emu.get_option(emu.OPT_BUCKET_TILES)
    emu.set_option(emu.OPT_BUCKET_TILES, tiles)
    try:
        for shape in ((2, 9, 2, 3, 2, 10, 21), (1, 41, 4, 7, 2, 50, 130), (1, 64, 2, 32, 2, 96, 320)):
            check(emu.Layout(emu.Model(*shape), 2, 1, 7, dtype), SIZES)
    finally:
        emu.set_option(emu.OPT_BUCKET_TILES, old)


@pytest.mark.gpu
@pytest.mark.parametrize("k", range(len(LARGE)))
def test_pieces_written_through(gpu_lib, k):
    shape, pad, dtype, sizes = LARGE[k]
    check(emu.Layout(emu.Model(*shape), 2, 1, pad, dtype), sizes)
