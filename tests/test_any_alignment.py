"""Segments whose rows start at any element: bit-exact against the oracle at the widths where the unit
arithmetic of the kernel can go wrong, and their tile counts against one tile per slice of a row."""
import random

import pytest

import oracle
from paper_2609_34645_amd import emu

# Row widths in elements of the row-parallel slices (o and down) at tp = 2: below, at and just above one
# 16-byte unit in both element types; around the 2 KB from which rows sit on the 128-byte grid; around one
# and two 4 KB tiles.
WIDTHS = [1, 3, 4, 5, 7, 8, 9, 13, 127, 511, 513, 1023, 1025, 2045, 2047, 2051, 4099]
PAIRS = [("bf16", "bf16"), ("fp32", "fp32"), ("fp32", "bf16"), ("bf16", "fp32")]


def _model(width, hidden=12, vocab=64):
    # query heads x head_dim = 2 * width (head_dim = width, one KV head per rank), MLP = 2 * width
    return emu.Model(1, hidden, 2, width, 2, 2 * width, vocab)


def through_groups(plan):
    """Tensor groups with which one launch moves the 1 GiB from which plans write through."""
    return -(-(1 << 30) // (plan.info["bytes_read"] + plan.info["bytes_written"]))


def run_through(plan, ws, S, D):
    """A reshard that has streamed, again as one launch of many groups that all name the same tensors, so that it
    writes through: D, refilled, must come out as it was, with the bytes around its tensors untouched."""
    import torch
    from gpu_util import Guard

    want = [t.clone() for t in D.tensors]
    for b in D.bufs:
        b.fill_(0xA5)
    g = Guard(keep=S.tensors, fills=[(D.tensors, 0xA5)], label="written through")
    n = through_groups(plan)
    plan.reshard_groups(ws, S.ptrs.repeat(n), D.ptrs.repeat(n))
    torch.cuda.synchronize()
    g.check()
    for i, (t, w) in enumerate(zip(D.tensors, want)):
        assert torch.equal(t, w), f"written through: destination tensor {i} differs"


def through_plan(width, a, b, pair):
    """A plan that writes through in enough groups. A copy: at odd widths throughout. A conversion: aligned but for
    o's and down's column slices, under a tenth of its bytes (more misaligned ones stream at any size)."""
    if pair[0] == pair[1]:
        m = _model(width, 9 if width > 2000 else 11, 512)
    else:
        m = _model(width, 64, 64 * (width // 3 + 8))
    return emu.Plan(emu.Layout(m, a, 1, 0, pair[0]), emu.Layout(m, b, 1, 48, pair[1]))


@pytest.mark.gpu
@pytest.mark.parametrize("tile_vecs", [0, 1, 16])
@pytest.mark.parametrize("pair", PAIRS, ids=lambda p: "-".join(p))
def test_widths_around_units_and_tiles(gpu_lib, pair, tile_vecs):
    """Split and Merge over TP at every width, into destinations whose surroundings must not change."""
    import torch
    from gpu_util import Guard, check_reshard, full_model, o_layout, upload_shards

    old = emu.get_option(emu.OPT_TILE_VECS)
    emu.set_option(emu.OPT_TILE_VECS, tile_vecs)
    try:
        for width in WIDTHS:
            m = _model(width, 9 if width > 2000 else 12)
            for a, b in ((1, 2), (2, 1)):
                src, dst = emu.Layout(m, a, 1, 0, pair[0]), emu.Layout(m, b, 1, 48, pair[1])
                plan = emu.Plan(src, dst)
                ws = plan.workspace()
                S, D = plan.alloc(0, fill=0x5A, guard=256), plan.alloc(1, fill=0xA5, guard=256)
                os_ = o_layout(src)
                upload_shards(oracle.shard(full_model(os_.model, width, pair[0]), os_), S, tp=a)
                g = Guard(keep=S.tensors, fills=[(D.tensors, 0xA5)], label=f"width {width} TP{a}->TP{b}")
                plan.reshard(ws, S.ptrs, D.ptrs)
                torch.cuda.synchronize()
                g.check()
                check_reshard(plan, S, D, label=f"width {width} {pair} TP{a}->TP{b}")
    finally:
        emu.set_option(emu.OPT_TILE_VECS, old)


@pytest.mark.gpu
@pytest.mark.parametrize("tile_vecs", [0, 1, 2, 8, 16])
@pytest.mark.parametrize("pair", PAIRS, ids=lambda p: "-".join(p))
def test_widths_written_through(gpu_lib, pair, tile_vecs):
    """The same widths written through, against the streaming result."""
    import torch

    old = emu.get_option(emu.OPT_TILE_VECS)
    emu.set_option(emu.OPT_TILE_VECS, tile_vecs)
    g = torch.Generator(device="cuda")
    g.manual_seed(tile_vecs)
    try:
        for width in WIDTHS:
            for a, b in ((1, 2), (2, 1)):
                plan = through_plan(width, a, b, pair)
                ws = plan.workspace()
                S, D = plan.alloc(0, guard=256), plan.alloc(1, fill=0xA5, guard=256)
                for x in S.bufs:
                    x.copy_(torch.randint(0, 256, x.shape, generator=g, device="cuda", dtype=torch.uint8))
                plan.reshard(ws, S.ptrs, D.ptrs)
                run_through(plan, ws, S, D)
    finally:
        emu.set_option(emu.OPT_TILE_VECS, old)


def test_no_more_tiles_than_slices_of_rows():
    """A plan takes no more tiles than one per tile-sized slice of each row, so that no plan outgrows a
    limit on its tables for the sake of its alignment; and every odd width is on the general path."""
    rng = random.Random(9)
    seen = 0
    for n in range(150):
        width = rng.choice(WIDTHS + [rng.randint(1, 5000)])
        m = emu.Model(rng.randint(1, 3), rng.randint(3, 60), 2, width, 2, 2 * width, rng.randint(8, 90))
        sdt, ddt = rng.choice(PAIRS)
        src, dst = emu.Layout(m, rng.choice([1, 2]), 1, 8, sdt), emu.Layout(m, rng.choice([1, 2]), 1, 8, ddt)
        kw = rng.choice([{}, dict(bucket_bytes=4 * rng.randint(2, 9000)), dict(src_bucket_bytes=4 * rng.randint(2, 9000))])
        plan = emu.Plan(src, dst, **kw)
        tb = plan.info["tile_bytes"]
        segs = plan.segments()
        assert plan.info["n_tiles"] <= sum(g["rows"] * -(-g["run"] // tb) for g in segs), (n, kw)
        odd = [g for g in segs if (g["dst_offset"] | g["run"]) % 16]
        assert plan.info["n_general_segments"] >= len(odd)
        seen += len(odd)
    assert seen > 500
