"""How calls are launched (stores' cache policy, workgroups resident per CU) on either side of each line of the
rules, read through a probe linked to the built library. No GPU needed."""
import contextlib
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2609_34645_amd import build, emu

HERE = os.path.dirname(os.path.abspath(__file__))
PLAIN, NT, THROUGH = 0, 1, 2
ONE_B = (16, 2048, 32, 64, 8, 8192, 128256)
RAGGED = (12, 996, 12, 83, 6, 2658, 50257)


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ is not available")
    if not os.path.exists(emu.LIB_PATH):
        build.build()
    emu.load()
    so = str(tmp_path_factory.mktemp("probe") / "probe.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(HERE, "launch_rules_probe.cpp"), emu.LIB_PATH, f"-Wl,-rpath,{build.PKG}", "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.probe_reshard.argtypes = [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_void_p]
    lib.probe_bucket.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_uint64, ctypes.c_int32, ctypes.c_void_p]
    lib.probe_reshard.restype = lib.probe_bucket.restype = None
    return lib


@contextlib.contextmanager
def options(**kw):
    keys = {getattr(emu, "OPT_" + k): v for k, v in kw.items()}
    old = {k: emu.get_option(k) for k in keys}
    try:
        for k, v in keys.items():
            emu.set_option(k, v)
        yield
    finally:
        for k, v in old.items():
            emu.set_option(k, v)


def plan(shape, src, dst, sdt="bf16", ddt="bf16", pads=(0, 0), **kw):
    m = emu.Model(*shape)
    return emu.Plan(emu.Layout(m, *src, pads[0], sdt), emu.Layout(m, *dst, pads[1], ddt), **kw)


def reshard(probe, p, groups=1):
    out = (ctypes.c_int32 * 3)()
    probe.probe_reshard(p._h, groups, out)
    return tuple(out)[:2]


def in_blocks(probe, p):
    out = (ctypes.c_int32 * 3)()
    probe.probe_reshard(p._h, 1, out)
    return bool(out[2])


def bucket(probe, p, B, unpack, side=0):
    out = (ctypes.c_int32 * 2)()
    probe.probe_bucket(p._h, side, B, int(unpack), out)
    return tuple(out)


def test_reshard_by_bytes_moved(probe):
    """Large transfers write through, small ones do not, and the groups of one launch count together."""
    big, small = plan(ONE_B, (4, 1), (2, 1)), plan((2, 256, 4, 64, 2, 688, 1024), (1, 1), (2, 1))
    assert reshard(probe, big) == (THROUGH, 12) and reshard(probe, small) == (NT, 12)
    moved = small.info["bytes_read"] + small.info["bytes_written"]
    n = -(-(1 << 30) // moved)
    assert reshard(probe, small, n - 1) == (NT, 12) and reshard(probe, small, n) == (THROUGH, 12)
    with options(NONTEMPORAL=0):
        assert reshard(probe, big) == (PLAIN, 12)
        assert reshard(probe, plan(ONE_B, (4, 1), (2, 1), "fp32", "bf16")) == (PLAIN, 6)
        assert reshard(probe, plan(ONE_B, (4, 1), (2, 1), "bf16", "fp32")) == (PLAIN, 14)
    with options(WG_PER_CU=7):
        assert reshard(probe, big) == (THROUGH, 7)


@pytest.mark.parametrize("pair, few, many", [(("fp32", "bf16"), (THROUGH, 6), (NT, 10)),
                                             (("bf16", "fp32"), (THROUGH, 14), (NT, 12))], ids=["narrow", "widen"])
def test_conversions_by_share_of_misaligned_bytes(probe, pair, few, many):
    """One misaligned segment does not change how the rest of a large converting plan is launched: the share of
    misaligned bytes decides, from an eighth on. Zero fill has no share, aligned or not."""
    assert reshard(probe, plan(ONE_B, (4, 1), (2, 1), *pair)) == few
    # o's slices of 66 columns per rank: 0.6% of the bytes
    p = plan((6, 4096, 4, 66, 4, 11008, 32000), (4, 1), (2, 1), *pair)
    assert p.info["n_general_segments"] > 0 and reshard(probe, p) == few
    # tensors of odd sizes, and zero fill that starts between vectors: 5%
    p = plan((6, 4098, 32, 64, 8, 11008, 32001), (4, 1), (4, 1), *pair, (8, 16))
    assert p.info["n_general_segments"] > 0 and p.info["zero_fill_bytes"] > 0 and reshard(probe, p) == few
    assert reshard(probe, plan((6, 4096, 32, 64, 8, 11004, 32000), (4, 1), (2, 1), *pair)) == many  # down: 22%
    assert reshard(probe, plan(RAGGED, (2, 1), (1, 2), *pair, (64, 64))) == many


@pytest.mark.parametrize("tile_vecs, copy, narrow, widen", [(1, 0, 24, 0), (2, 24, 12, 28), (8, 6, 4, 7), (16, 3, 4, 4)])
def test_residency_at_other_tile_sizes(probe, tile_vecs, copy, narrow, widen):
    """The bytes in flight that 4 KB tiles run best with, but not fewer than 4 of the larger tiles in conversions."""
    with options(TILE_VECS=tile_vecs):
        assert reshard(probe, plan(ONE_B, (4, 1), (2, 1)))[1] == copy
        assert reshard(probe, plan(ONE_B, (4, 1), (2, 1), "fp32", "bf16"))[1] == narrow
        assert reshard(probe, plan(ONE_B, (4, 1), (2, 1), "bf16", "fp32"))[1] == widen


def test_tiles_that_end_inside_a_granule(probe):
    """Buckets whose size is a multiple of a vector but not of 64 bytes put most of a fused plan's tiles off the
    granule; a size that is keeps them on it, at any phase of a 128-byte line."""
    for pair, cap in ((("bf16", "bf16"), (12, 12)), (("fp32", "bf16"), (6, 6)), (("bf16", "fp32"), (14, 12))):
        for B, want in (((1 << 26) - 64, (THROUGH, cap[0])), ((1 << 26) - 16, (NT, cap[1]))):
            p = plan(ONE_B, (4, 1), (2, 1), *pair, bucket_bytes=B)
            assert p.info["n_general_segments"] == 0 and reshard(probe, p) == want, (pair, B)
    # row slices off the granule, 22% of the bytes in the Merge: copies still write through, conversions do not;
    # in the Split each slice is a whole tensor
    shape = (6, 3144, 12, 20, 6, 10512, 52648)
    for pair, want in ((("bf16", "bf16"), THROUGH), (("fp32", "bf16"), NT), (("bf16", "fp32"), NT)):
        assert reshard(probe, plan(shape, (2, 1), (1, 1), *pair))[0] == want
        assert reshard(probe, plan(shape, (1, 1), (2, 1), *pair))[0] == THROUGH


def test_order_by_tiles(probe):
    """Maps of fewer than four rounds of blocks go in contiguous eighths, unless some of their tiles are misaligned."""
    for vocab, blocks in ((4 * 32 * 1024 - 1000, False), (4 * 32 * 1024, True)):
        p = plan((1, 64, 2, 32, 2, 64, vocab), (1, 1), (1, 1), pads=(0, 96))
        assert (p.info["n_tiles"] >= 8192) == blocks and in_blocks(probe, p) == blocks
    assert not in_blocks(probe, plan((6, 256, 8, 32, 4, 864, 1024), (2, 1), (1, 1)))
    p = plan((6, 250, 8, 32, 4, 864, 1024), (2, 1), (1, 1))
    assert p.info["n_general_segments"] > 0 and p.info["n_tiles"] < 8192 and in_blocks(probe, p)


def test_write_through_without_a_cap(probe):
    big, wide = plan(ONE_B, (4, 1), (2, 1)), plan(ONE_B, (4, 1), (2, 1), "bf16", "fp32")
    with options(WG_PER_CU=0):
        assert reshard(probe, big) == reshard(probe, wide) == (THROUGH, 0)
        assert bucket(probe, big, 1 << 28, False) == bucket(probe, big, 1 << 28, True) == (THROUGH, 0)
    with options(TILE_VECS=1):
        assert reshard(probe, plan(ONE_B, (4, 1), (2, 1))) == (THROUGH, 0)
        assert reshard(probe, plan(ONE_B, (4, 1), (2, 1), "bf16", "fp32")) == (NT, 0)


def test_tensors_off_the_grid(probe):
    """Buckets on the 4 KB grid, tensors off it: the unpack moves its chunks; the pack's loads start inside a dword in
    bf16 and on dwords in fp32."""
    for dtype, pack in (("bf16", 12), ("fp32", 10)):
        p = plan((10, 1997, 12, 66, 12, 7896, 6653), (3, 3), (3, 3), dtype, dtype, (8, 8))
        assert bucket(probe, p, 1 << 22, False)[1] == pack and bucket(probe, p, 1 << 22, True)[1] == 12
        assert bucket(probe, p, (1 << 22) + 4, False)[1] == bucket(probe, p, (1 << 22) + 4, True)[1] == 12


def test_buckets_by_set_size(probe):
    big = plan(ONE_B, (4, 1), (4, 1))
    for unpack in (False, True):
        assert bucket(probe, big, 1 << 28, unpack) == (THROUGH, 10)
        assert bucket(probe, big, (1 << 28) - 2, unpack) == (THROUGH, 12)
        with options(NONTEMPORAL=0):
            assert bucket(probe, big, 1 << 28, unpack) == (PLAIN, 10)
    for layers, policy in ((3, NT), (4, THROUGH)):  # sets of 266 and 288 MB: from 2^28 bytes on, whatever the buckets
        p = plan((layers, 996, 12, 83, 6, 2658, 50257), (2, 1), (2, 1), pads=(64, 64))
        assert (p.info["src_bytes"] >= 1 << 28) == (policy == THROUGH)
        for unpack in (False, True):
            assert bucket(probe, p, 1 << 22, unpack)[0] == bucket(probe, p, (1 << 22) + 2, unpack)[0] == policy


def test_the_write_through_tests_write_through(probe):
    """The plans and sets that the bit-exact tests of writing through run are launched so."""
    import test_any_alignment as t
    from test_bucket_pieces import LARGE

    for tile_vecs in (0, 1, 2, 8, 16):
        with options(TILE_VECS=tile_vecs):
            for width in t.WIDTHS:
                for pair in t.PAIRS:
                    for a, b in ((1, 2), (2, 1)):
                        p = t.through_plan(width, a, b, pair)
                        n = t.through_groups(p)
                        assert n <= 65535 and (p.info["n_general_segments"] > 0 or width in (4, 8))
                        if (pair, tile_vecs) != (("bf16", "fp32"), 1):  # streams, see reshard_rule
                            assert reshard(probe, p, n)[0] == THROUGH, (width, pair, tile_vecs)
    for shape, pad, dtype, sizes in LARGE:
        lay = emu.Layout(emu.Model(*shape), 2, 1, pad, dtype)
        p = emu.Plan(lay, lay)
        assert all(bucket(probe, p, B, unpack)[0] == THROUGH for B in sizes for unpack in (False, True)), (shape, dtype)
