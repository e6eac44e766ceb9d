// How one reshard, pack or unpack call is launched, from what it moves: the cache policy of its stores,
// the most workgroups resident per CU and the order of the reshard's tiles. Host code of its own, so that the
// rules can be checked without a GPU.
#include "emu.h"
#include "emu_internal.h"

namespace emu {

// Residency bounds the bytes in flight per CU: on MI355X a copy stream runs fastest with about 24-48 KB in
// flight per CU and drops by about 8% at 128 KB, where the HBM read/write mix degrades. Automatic (-1):
// flight / tile_bytes workgroups, at least `least`, and no cap from 32 up, with `flight` in destination bytes.
static int resident(uint64_t tile_bytes, uint64_t flight, int least = 2) {
  const int64_t set = option(EMU_OPT_WG_PER_CU);
  if (set >= 0) return int(set);
  const int64_t cap = int64_t(flight / (tile_bytes ? tile_bytes : 1));
  return cap < least ? least : cap >= 32 ? 0 : int(cap);
}

// The reshard. Measured at 4 KB tiles, several settings in one process on the same buffers, with the states
// in rotation that no cache holds:
//  - Residency (flight, destination bytes in flight per CU). Copies: 48 KB; 8 / 10 / 12 / 14 tiles ran the 1B
//    TP4 -> TP2 reshard in 912 / 890 / 890 / 900 us and a decoder with odd widths in 155 / 147 / 145 / 148.
//    fp32 -> bf16, which reads twice what it writes: 24 KB; 4 / 6 / 8 / 10 tiles took 1548 / 1319 / 1340 / 1355 us
//    on aligned 1B shards. From an eighth of the bytes at any alignment on 40 KB: with 6 tiles a first pass over new
//    buffers takes 250 us against 241 (odd widths, 1.4 GB) and sets of 23 and 36 MB 6.2 and 7.9 against 5.7 and 7.5,
//    more than the 211 against 215 us that later passes gain. bf16 -> fp32, which reads half: written through 56 KB,
//    12 / 14 / 16 tiles in 1377 / 1364 / 1372 us (1B, fused to separate formats), with plain stores 56 KB, 10 / 12 /
//    14 / 16 in 1623 / 1498 / 1459 / 1461, streaming 48 KB, in 1414 / 1382 / 1394 / 1418.
//    Conversions keep at least 4 of the larger tiles: 2 / 4 / 6 took 1895 / 1378 / 1447 us at 8 KB (fp32 -> bf16),
//    1776 / 1473 / 1527 at 16 KB, and 1637 / 1391 / 1447 for bf16 -> fp32 at 16 KB. Copies at 16 KB run best with
//    2: 929 / 974 / 1009.
//  - Cache policy. Writing through gains from about 1 GB moved per launch on (1B copy 890 against 914 us, 8B 4823
//    against 4928, fp32 -> bf16 1319 against 1335, bf16 -> fp32 1364 against 1382; copies with units at any alignment:
//    odd widths, 4.8 GB, 724 against 743, 8B into and out of odd buckets 10.12 against 10.28 ms), not below (0.7 GB:
//    107.2 against 105.5; 4 MB: 2.7 against 2.5). Conversions at any alignment: written through
//    / streaming, fp32 -> bf16 at a share of 0 / 0.006 / 0.22 / 0.67 / 0.8 of the bytes 1070 / 1079, 992 / 1002, 1089 /
//    1088, 1113 / 1096 and 447 / 443 us; bf16 -> fp32 at 0 / 0.006 / 0.22 / 0.67: 1104 / 1108, 1017 / 1028, 1119 /
//    1116 and 1133 / 1127. Widening at 1 KB tiles streams: 1601 us against 1635.
//    Tiles that end inside a 64-byte granule (whole vectors, but destination offsets or strides off the granule) are
//    written to memory in two parts, where streaming stores meet in the L2. Copies at such a share of 0.18 / 0.22 /
//    0.28 / 0.28 / 0.48 / 0.60: 464 / 467, 588 / 588, 455 / 461, 950 / 936, 973 / 931 and 629 / 591, 8B into buckets
//    of 2^28 - 16 bytes (0.6) 5,514 / 5,030. fp32 -> bf16 at 0.06 / 0.18 / 0.22 / 0.28 / 0.48: 651 / 648, 701 / 679,
//    881 / 844, 1,466 / 1,356 and 1,508 / 1,359; bf16 -> fp32 at 0.06 / 0.11 / 0.18 / 0.22 / 0.44: 670 / 668, 1,443 /
//    1,416, 716 / 697, 908 / 878 and 1,584 / 1,455. So copies write through up to a third, conversions up to a tenth,
//    bytes at any alignment counted in.
//  - Order. Blocks of kReshardBlock tiles from four rounds over the XCDs on (8,192 tiles), contiguous eighths of the
//    map below, where the front of one to three rounds leaves XCDs idle at its end: three states in rotation, in
//    blocks / eighths, 2,789 tiles 5.28 / 4.72 us, 3,371 tiles 6.45 / 6.04, 5,321 tiles 9.04 / 8.62, 7,009 tiles 11.05 /
//    11.03, 10,385 tiles 15.3 / 15.1 (a Merge 15.6 / 15.9), 17,137 tiles 23.5 / 23.7. Tiles at any alignment take longer
//    than others, and eighths deal them unevenly: blocks there, 7,945 tiles 13.55 / 13.95, 8,000 tiles 12.8 / 13.2.
constexpr uint64_t kThroughBytes = 1ull << 30;  // read and written by one reshard launch
constexpr uint64_t kBlockTiles = 4 * kXcdCount * kReshardBlock;

LaunchRule reshard_rule(const Plan& P, uint32_t groups) {
  const uint64_t moved = (P.info.bytes_read + P.info.bytes_written) * groups;
  const uint64_t written = P.info.bytes_written;
  const bool thin = P.cvt == CVT_BF16_F32 && P.tile_vecs == 1;
  const bool whole = P.cvt == CVT_NONE ? P.off_bytes <= written / 3 : P.any_bytes + P.off_bytes <= written / 10;
  int policy = POL_PLAIN;
  if (option(EMU_OPT_NONTEMPORAL) != 0) policy = moved >= kThroughBytes && whole && !thin ? POL_THROUGH : POL_NT;
  uint64_t flight = 48 << 10;
  if (P.cvt == CVT_F32_BF16) flight = (P.any_bytes < written / 8 ? 24 : 40) << 10;
  else if (P.cvt == CVT_BF16_F32 && policy != POL_NT) flight = 56 << 10;
  return {policy, resident(P.tile_bytes, flight, P.cvt == CVT_NONE ? 2 : 4), P.ws.n_map >= kBlockTiles || P.any_bytes > 0};
}

// Pack and unpack cut chunks on the stream's grid unless the destination's differs: buckets whose size is not
// a multiple of 4 KB (pack), tensors at stream offsets that are not (unpack).
bool chunks_realign(const SideInfo& s, uint64_t B, bool unpack) {
  return unpack ? !s.offsets_grid : B % kTileChunkBytes != 0;
}

// Pack and unpack, residency and cache policy as for the reshard. 10 / 12 / 16 chunks per CU: 9,537 / 9,738 /
// 10,087 us for the 8B pack and unpack, whose chunks end on tensor and bucket ends; 298 / 288 / 292 us where
// chunks are moved to the destination's grid and hold several pieces (odd widths). Buckets that start inside a
// dword make the unpack's loads slower: 12 per CU there too (8B at 2^28 - 2: 4,838 us against 4,943 at 10; at
// 2^28 - 4: 4,792 against 4,797), and tensors that do the pack's, whatever the buckets (odd widths in 4 MB buckets,
// 2.3 GB: 708 us against 722; at tensors off the 4 KB grid, but on dwords, 715 against 702).
//
// Written through / streaming. Sets in rotation that no cache holds, buckets on the 4 KB grid, unpack: 10.97 /
// 10.84 us (a set of 26 MB), 40.1 / 41.6 (128), 95.3 / 98.8 (317), 901 / 936 (3.0 GB, pack 900 / 941). Other bucket
// sizes, where pieces stored under lane masks lose what the others gain: 39.0 / 39.0 (120 MB), 65.3 / 65.2 (207, pack
// 65.9 / 65.6), 91.7 / 91.9 (295, pack 92.2 / 92.3), 174 / 176 (557). The same set again and again, part of which the
// last-level cache keeps, streams better below the line: pack 40.9 / 40.3 (125 MB), unpack 59.6 / 58.2 (190 MB in
// tensors of 86 KB), 75.9 / 73.9 (235).
constexpr uint64_t kThroughBucketBytes = 1ull << 29;  // read and written by one pack or unpack

LaunchRule bucket_rule(const SideInfo& s, uint64_t B, bool unpack) {
  const bool shifted = chunks_realign(s, B, unpack) || B % 4 != 0 || !s.offsets_dword;
  int policy = POL_PLAIN;
  if (option(EMU_OPT_NONTEMPORAL) != 0) policy = 2 * s.total_bytes >= kThroughBucketBytes ? POL_THROUGH : POL_NT;
  return {policy, resident(kTileChunkBytes, (shifted ? 48 : 40) << 10), true};
}

}  // namespace emu
