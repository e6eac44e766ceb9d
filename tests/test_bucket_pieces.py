"""Pack and unpack of pieces at every length and phase: against each rank's stream, put together by torch."""
import pytest

from paper_2609_34645_amd import emu

# Bucket sizes: a few elements; around one and two units of 16 bytes; around a 4 KB chunk, with odd sizes that
# put bucket k at any phase; larger than any stream (the division by the bucket size at its extremes)
SIZES = [4, 12, 16, 20, 28, 44, 4092, 4096, 4100, 6140, 12292, (1 << 33) + 4, 1 << 63]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("tiles", [1, 0], ids=["tile_per_wg", "persistent"])
def test_pieces(gpu_lib, dtype, tiles):
    import torch
    from gpu_util import Guard

    old = emu.get_option(emu.OPT_BUCKET_TILES)
    emu.set_option(emu.OPT_BUCKET_TILES, tiles)
    try:
        for shape in ((2, 9, 2, 3, 2, 10, 21), (1, 41, 4, 7, 2, 50, 130), (1, 64, 2, 32, 2, 96, 320)):
            lay = emu.Layout(emu.Model(*shape), 2, 1, 7, dtype)
            plan = emu.Plan(lay, lay)
            ws = plan.workspace()
            S = plan.alloc(0, guard=64)
            g = torch.Generator(device="cuda")
            g.manual_seed(shape[1])
            for b in S.bufs:
                b.copy_(torch.randint(0, 256, b.shape, generator=g, device="cuda", dtype=torch.uint8))
            ranks = {}
            for d, t in zip(plan.tensors(0), S.tensors):
                ranks.setdefault(d["rank"], []).append(t)
            streams = {r: torch.cat(ts) for r, ts in ranks.items()}
            for B in SIZES:
                bufs, bptrs = plan.alloc_buckets(0, B, fill=0xA5, guard=64)
                R = plan.alloc(0, fill=0x5A, guard=64)
                guard = Guard(keep=S.tensors, fills=[(bufs, 0xA5), (R.tensors, 0x5A)], label=f"{shape} B={B}")
                plan.pack(ws, 0, B, S.ptrs, bptrs)
                plan.unpack(ws, 0, B, bptrs, R.ptrs)
                torch.cuda.synchronize()
                guard.check()
                for i, b in zip(plan.bucket_info(0, B), bufs):
                    want = streams[i["rank"]][i["stream_offset"]:i["stream_offset"] + i["bytes"]]
                    assert torch.equal(b, want), (shape, B, i)
                for i, (s, r) in enumerate(zip(S.tensors, R.tensors)):
                    assert torch.equal(s, r), (shape, B, i)
    finally:
        emu.set_option(emu.OPT_BUCKET_TILES, old)
