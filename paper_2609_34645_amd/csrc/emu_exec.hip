// Device side of the EMU reshard library for CDNA4 (gfx950): the reshard kernel that executes a
// compiled copy map, the bucket pack/unpack kernel, the small kernels that build a plan's tile map and
// bucket stream tables in its workspace at upload, and the C ABI entry points that launch them.
//
// Both kernels are pure HBM streams: no arithmetic on the data (fp32 <-> bf16 conversion aside),
// integer address math only. Every thread moves 16-byte vectors, from and to any element address, a tile is
// threads * U vectors, and all U loads of a tile are issued before its stores. How many tiles are
// resident per CU is bounded (EMU_OPT_WG_PER_CU), so that each CU keeps 24-56 KB of tiles in flight:
// enough to cover HBM latency, and few enough that the mixed read/write stream does not congest. Both
// tile kernels run one wave64 per workgroup, so that each tile's address computation (map entry,
// descriptor or rank record, pointers) is done once rather than once per wave.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "emu_internal.h"


namespace emu {

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------------
// device helpers
// ------------------------------------------------------------------------------------------------

// Global-address-space views: table-loaded pointers are generic to the compiler, which would emit
// flat loads; casting to address space 1 gives global_load/store_dwordx4 with a scalar base.
typedef __attribute__((address_space(1))) v4u gv4u;
typedef __attribute__((address_space(1))) uint8_t gu8;

// Cache policies of the kernels' loads and stores (enum Policy). POL_NT and POL_THROUGH load with "nt" (streaming).
// POL_NT also stores with it; POL_THROUGH stores with "sc1 nt", as buffer stores: written through to memory
// as they come, instead of staying in the XCD's L2 until evicted. With as many tiles in flight as the
// reshard needs to cover its tables' latency, write-through holds HBM's read/write mix better: a bare
// 4 KB-tile copy of 8 GB at 8 / 10 resident waves per CU ran at 6.71 / 6.55 TB/s against 6.52 / 6.28 with
// "nt" (6.80 / 6.73 at 6), the 8B reshard at 10 per CU in 4.80 ms against 4.93. Which call takes which:
// emu_launch.cpp.
constexpr int kThroughBits = 2 | 16;  // nt | sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t whole_range(uint8_t* base) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000);  // raw, unswizzled, 2^32 - 1 bytes
}

template <int POL>
__device__ __forceinline__ v4u ld16(const uint8_t* base, uint32_t off) {
  const gv4u* p = (const gv4u*)((const gu8*)base + off);
  if constexpr (POL != POL_PLAIN) return __builtin_nontemporal_load(p);
  else return *p;
}

template <int POL>
__device__ __forceinline__ void st16(uint8_t* base, uint32_t off, v4u v) {
  if constexpr (POL == POL_THROUGH) __builtin_amdgcn_raw_buffer_store_b128(v, whole_range(base), off, 0, kThroughBits);
  else if constexpr (POL == POL_NT) __builtin_nontemporal_store(v, (gv4u*)((gu8*)base + off));
  else *(gv4u*)((gu8*)base + off) = v;
}

__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) v2u gv2u;

template <int POL>
__device__ __forceinline__ v2u ld8(const uint8_t* base, uint32_t off) {
  const gv2u* p = (const gv2u*)((const gu8*)base + off);
  if constexpr (POL != POL_PLAIN) return __builtin_nontemporal_load(p);
  else return *p;
}

template <int POL>
__device__ __forceinline__ void st8(uint8_t* base, uint32_t off, v2u v) {
  if constexpr (POL == POL_THROUGH) __builtin_amdgcn_raw_buffer_store_b64(v, whole_range(base), off, 0, kThroughBits);
  else if constexpr (POL == POL_NT) __builtin_nontemporal_store(v, (gv2u*)((gu8*)base + off));
  else *(gv2u*)((gu8*)base + off) = v;
}

// The same at any element (2-byte) address. gfx950 moves 16 bytes per lane from and to any byte address in
// one instruction; lanes that cover a contiguous span cost one more cache line per instruction. A copy of
// 4 GB from a source 2 bytes off ran at 6.51 TB/s, 4 or 8 bytes off at 6.62, to a destination 2 bytes off at
// 6.66, aligned on both sides at 6.68 (each at its best residency from 8 per CU up), so no realignment in
// registers is needed.
typedef v4u v4u_any __attribute__((aligned(2)));
typedef v2u v2u_any __attribute__((aligned(2)));

template <int POL>
__device__ __forceinline__ v4u ld16_any(const uint8_t* base, uint32_t off) {
  const auto* p = (const __attribute__((address_space(1))) v4u_any*)((const gu8*)base + off);
  if constexpr (POL != POL_PLAIN) return __builtin_nontemporal_load(p);
  else return *p;
}

template <int POL>
__device__ __forceinline__ void st16_any(uint8_t* base, uint32_t off, v4u v) {
  auto* p = (__attribute__((address_space(1))) v4u_any*)((gu8*)base + off);
  if constexpr (POL != POL_PLAIN) __builtin_nontemporal_store(v, p);
  else *p = v;
}

template <int POL>
__device__ __forceinline__ v2u ld8_any(const uint8_t* base, uint32_t off) {
  const auto* p = (const __attribute__((address_space(1))) v2u_any*)((const gu8*)base + off);
  if constexpr (POL != POL_PLAIN) return __builtin_nontemporal_load(p);
  else return *p;
}

template <int POL>
__device__ __forceinline__ void st8_any(uint8_t* base, uint32_t off, v2u v) {
  auto* p = (__attribute__((address_space(1))) v2u_any*)((gu8*)base + off);
  if constexpr (POL != POL_PLAIN) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// fp32 bits -> bf16 bits: round to nearest, ties to even; a NaN keeps its sign and top payload bits and
// gets the quiet bit (so that a NaN whose payload sits in the low half never turns into infinity).
__device__ __forceinline__ uint32_t bf16_rne(uint32_t u) {
  const uint32_t r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  return (u & 0x7fffffffu) > 0x7f800000u ? ((u >> 16) | 0x40u) : r;
}

// Source data behind one 16-byte destination vector, per element conversion of the plan:
// CVT_NONE one 16-byte vector; CVT_F32_BF16 two (8 fp32 -> 8 bf16); CVT_BF16_F32 half of one (4 bf16).
template <int CVT> struct Raw { v4u a; };
template <> struct Raw<CVT_F32_BF16> { v4u a, b; };
template <> struct Raw<CVT_BF16_F32> { v2u a; };

template <int CVT>
constexpr uint32_t kSrcVecBytes = CVT == CVT_F32_BF16 ? 32u : CVT == CVT_BF16_F32 ? 8u : 16u;

template <int CVT, int POL>
__device__ __forceinline__ Raw<CVT> ld_raw(const uint8_t* s, uint32_t off) {
  Raw<CVT> r;
  if constexpr (CVT == CVT_F32_BF16) {
    r.a = ld16<POL>(s, off);
    r.b = ld16<POL>(s, off + 16u);
  } else if constexpr (CVT == CVT_BF16_F32) {
    r.a = ld8<POL>(s, off);
  } else {
    r.a = ld16<POL>(s, off);
  }
  return r;
}

template <int CVT>
__device__ __forceinline__ v4u cook(const Raw<CVT>& r) {
  if constexpr (CVT == CVT_F32_BF16) {
    v4u o;
    o.x = bf16_rne(r.a.x) | (bf16_rne(r.a.y) << 16);
    o.y = bf16_rne(r.a.z) | (bf16_rne(r.a.w) << 16);
    o.z = bf16_rne(r.b.x) | (bf16_rne(r.b.y) << 16);
    o.w = bf16_rne(r.b.z) | (bf16_rne(r.b.w) << 16);
    return o;
  } else if constexpr (CVT == CVT_BF16_F32) {
    return v4u{r.a.x << 16, r.a.x & 0xffff0000u, r.a.y << 16, r.a.y & 0xffff0000u};
  } else {
    return r.a;
  }
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(x));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(x >> 32));
  return (uint64_t(hi) << 32) | lo;
}

// Ends the wait for all loads of a tile at once. Ahead of stores that a lane mask guards: the compiler
// counts loads and stores in one counter and cannot know which masked stores were issued, so without this
// it waits for the tile's first stores to complete before it issues the last ones. A tile without masked
// stores needs no such wait, which is why full tiles have paths of their own below. At 6 resident tiles per
// CU the 1B TP4 -> TP2 reshard took 957 us with both, 1,086 us before; at 8 per CU 926 against 962.
//
// The loaded values pass through the (empty) statements: a load that only a guarded store uses is otherwise
// moved into that store's block, behind the wait, where it takes a second memory latency. With a plain s_waitcnt
// here, reshard + pack + unpack of the tiny decoder (4 MB, replayed in a graph) took 14.4 us in bf16 and 17.6 in
// fp32; without any wait 13.3 and 15.9; this way 12.6 and 15.1.
__device__ __forceinline__ void arrived(v4u& a) { asm volatile("" : "+v"(a)); }
__device__ __forceinline__ void arrived(v2u& a) { asm volatile("" : "+v"(a)); }
template <int CVT>
__device__ __forceinline__ void arrived(Raw<CVT>& r) {
  arrived(r.a);
  if constexpr (CVT == CVT_F32_BF16) arrived(r.b);
}
template <typename T, int N>
__device__ __forceinline__ void loads_done(T (&r)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) arrived(r[k]);
}

// Workgroup-cooperative copy of n > 0 bytes between any even addresses (n < 2^31). The body runs in 16-byte
// units on the destination's 16-byte grid; the first and the last unit are moved inward to the copy's ends
// and overlap their neighbours, which write the same bytes there. P units per lane are in flight. m is the
// phase of d on the grid, known from the tables (tensors and buckets are 16-byte aligned), so that the loads
// need not wait for the destination's pointer.
template <int NTH, int P, int POL>
__device__ __forceinline__ void wg_copy(const uint8_t* __restrict__ s, uint8_t* __restrict__ d, uint32_t n, uint32_t m) {
  const uint32_t tid = threadIdx.x;
  constexpr uint32_t kFull = uint32_t(NTH) * P * 16u;
  if (n == kFull && m == 0) {
    v4u r[P];
#pragma unroll
    for (int k = 0; k < P; ++k) r[k] = ld16_any<POL>(s, (k * NTH + tid) * 16u);
#pragma unroll
    for (int k = 0; k < P; ++k) st16<POL>(d, (k * NTH + tid) * 16u, r[k]);
  } else if (n >= 16u) {
    const uint32_t cnt = (n + m + 15u) / 16u;
#pragma nounroll
    for (uint32_t b = 0; b < cnt; b += uint32_t(NTH) * P) {
      uint32_t at[P];
      v4u r[P];
#pragma unroll
      for (int k = 0; k < P; ++k) {
        const uint32_t x = umin(b + k * NTH + tid, cnt - 1) * 16u;
        at[k] = umin(x < m ? 0u : x - m, n - 16u);
        r[k] = ld16_any<POL>(s, at[k]);
      }
      loads_done(r);
#pragma unroll
      for (int k = 0; k < P; ++k)
        if (b + k * NTH + tid < cnt) st16_any<POL>(d, at[k], r[k]);
    }
  } else if (tid < n / 2u) {
    reinterpret_cast<uint16_t*>(d)[tid] = reinterpret_cast<const uint16_t*>(s)[tid];
  }
}

// ------------------------------------------------------------------------------------------------
// reshard kernel: one tile = kReshardThreads * U destination vectors of one segment
// ------------------------------------------------------------------------------------------------

#ifndef EMU_RESHARD_WAVES_PER_EU
#define EMU_RESHARD_WAVES_PER_EU 4
#endif
#ifndef EMU_BUCKET_WAVES_PER_EU
#define EMU_BUCKET_WAVES_PER_EU 4
#endif
#ifndef EMU_BUCKET_UNROLL
#define EMU_BUCKET_UNROLL 8
#endif
#ifndef EMU_BUCKET_TILE_VECS
#define EMU_BUCKET_TILE_VECS 4
#endif
#ifndef EMU_BUCKET_TILE_THREADS
#define EMU_BUCKET_TILE_THREADS 64
#endif
constexpr int kXcds = int(kXcdCount);  // workgroups are dealt to the XCDs round-robin
constexpr int kBucketUnroll = EMU_BUCKET_UNROLL;
constexpr int kBucketTileVecs = EMU_BUCKET_TILE_VECS;  // vectors per thread per pass of k_buckets_tile
constexpr int kBucketTileThreads = EMU_BUCKET_TILE_THREADS;  // workgroup size of k_buckets_tile

template <int U, bool LDS>
__device__ __forceinline__ void stage_through_lds(v4u (&r)[U], v4u* stage) {
  if constexpr (LDS) {
    const uint32_t tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < U; ++u) stage[u * kReshardThreads + tid] = r[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = stage[u * kReshardThreads + tid];
    __syncthreads();
  }
}

// Rows of rv vectors at strides ss and ds bytes from s and d, read in row-major vector order: the tile
// holds vectors r0 .. r0 + last of that order (FULL: as many as the tile has). Vector n is in row n / rv (a
// multiply-high by the host's magic number) at column n % rv; the host keeps every in-tile byte offset
// below 2^31.
template <int U, int POL, bool ZERO, bool LDS, int CVT, bool FULL>
__device__ __forceinline__ void tile_rows(const uint8_t* s, uint8_t* d, uint32_t r0, uint32_t last, uint32_t rv,
                                          uint32_t mg, uint32_t ss, uint32_t ds, v4u* stage) {
  const uint32_t tid = threadIdx.x;
  v4u r[U];
  if constexpr (ZERO) {
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = v4u{0, 0, 0, 0};
  } else {
    Raw<CVT> raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = u * kReshardThreads + tid, n = r0 + (FULL ? i : umin(i, last));
      const uint32_t q = rv > 1 ? __umulhi(n, mg) : n;
      raw[u] = ld_raw<CVT, POL>(s, q * ss + (n - q * rv) * kSrcVecBytes<CVT>);
    }
    if constexpr (!FULL) loads_done(raw);
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = cook<CVT>(raw[u]);
  }
  stage_through_lds<U, LDS>(r, stage);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = u * kReshardThreads + tid;
    const uint32_t n = r0 + i;
    const uint32_t q = rv > 1 ? __umulhi(n, mg) : n;
    if (FULL || i <= last) st16<POL>(d, q * ds + (n - q * rv) * 16u, r[u]);
  }
}

// A contiguous run of cnt (1 <= cnt <= kReshardThreads * U) destination vectors (FULL: as many as the tile has).
template <int U, int POL, bool ZERO, bool LDS, int CVT, bool FULL>
__device__ __forceinline__ void tile_run(const uint8_t* s, uint8_t* d, uint32_t cnt, v4u* stage) {
  const uint32_t tid = threadIdx.x;
  const uint32_t last = cnt - 1;
  v4u r[U];
  if constexpr (ZERO) {
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = v4u{0, 0, 0, 0};
  } else {
    Raw<CVT> raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = u * kReshardThreads + tid;
      raw[u] = ld_raw<CVT, POL>(s, (FULL ? i : umin(i, last)) * kSrcVecBytes<CVT>);
    }
    if constexpr (!FULL) loads_done(raw);
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = cook<CVT>(raw[u]);
  }
  stage_through_lds<U, LDS>(r, stage);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = u * kReshardThreads + tid;
    if (FULL || i <= last) st16<POL>(d, i * 16u, r[u]);
  }
}

// fp32 -> bf16 tiles, in source vectors: a tile of cnt destination vectors reads 2 * cnt source vectors
// of four fp32 each and writes 2 * cnt eight-byte halves. Each lane loads whole source vectors,
// consecutive across the lanes, and stores the four converted elements (8 bytes), so every load and
// every store instruction covers one contiguous span. Reading a destination vector's two source
// vectors in one lane instead makes every load instruction touch twice the cache lines it uses.
__device__ __forceinline__ v2u to_bf16x4(v4u a) {
  return v2u{bf16_rne(a.x) | (bf16_rne(a.y) << 16), bf16_rne(a.z) | (bf16_rne(a.w) << 16)};
}

// At most 8 destination vectors per lane per pass (16 source vectors, 64 VGPRs): larger tiles are moved in
// passes, so that the conversion never spills registers.
template <int U>
constexpr int kCvtPass = U > 8 ? 8 : U;

template <int U, int POL, bool FULL>
__device__ __forceinline__ void tile_run_f32_bf16(const uint8_t* s, uint8_t* d, uint32_t cnt) {
  constexpr int P = kCvtPass<U>;
  const uint32_t tid = threadIdx.x;
  const uint32_t last = 2 * cnt - 1;
#pragma unroll
  for (int h = 0; h < U / P; ++h) {
    v4u a[2 * P];
#pragma unroll
    for (int k = 0; k < 2 * P; ++k) {
      const uint32_t i = (h * 2 * P + k) * kReshardThreads + tid;
      a[k] = ld16<POL>(s, (FULL ? i : umin(i, last)) * 16u);
    }
    if constexpr (!FULL) loads_done(a);
#pragma unroll
    for (int k = 0; k < 2 * P; ++k) {
      const uint32_t i = (h * 2 * P + k) * kReshardThreads + tid;
      if (FULL || i <= last) st8<POL>(d, i * 8u, to_bf16x4(a[k]));
    }
  }
}

// The same rows converted: destination vectors r0 .. r0 + last, moved as halves (four fp32 read, four
// bf16 written). Half n of the tile belongs to destination vector r0 + n / 2, in row (r0 + n / 2) / rv;
// its column in halves is 2 r0 + n less twice the row's first vector.
template <int U, int POL, bool FULL>
__device__ __forceinline__ void tile_rows_f32_bf16(const uint8_t* s, uint8_t* d, uint32_t r0, uint32_t last,
                                                   uint32_t rv, uint32_t mg, uint32_t ss, uint32_t ds) {
  constexpr int P = kCvtPass<U>;
  const uint32_t tid = threadIdx.x;
  const uint32_t lasth = 2 * last + 1, h = 2 * rv;
#pragma unroll
  for (int p = 0; p < U / P; ++p) {
    v4u a[2 * P];
#pragma unroll
    for (int k = 0; k < 2 * P; ++k) {
      const uint32_t i = (p * 2 * P + k) * kReshardThreads + tid, n = 2 * r0 + (FULL ? i : umin(i, lasth));
      const uint32_t q = rv > 1 ? __umulhi(n >> 1, mg) : (n >> 1);
      a[k] = ld16<POL>(s, q * ss + (n - q * h) * 16u);
    }
    if constexpr (!FULL) loads_done(a);
#pragma unroll
    for (int k = 0; k < 2 * P; ++k) {
      const uint32_t i = (p * 2 * P + k) * kReshardThreads + tid;
      const uint32_t n = 2 * r0 + i;
      const uint32_t q = rv > 1 ? __umulhi(n >> 1, mg) : (n >> 1);
      if (FULL || i <= lasth) st8<POL>(d, q * ds + (n - q * h) * 8u, to_bf16x4(a[k]));
    }
  }
}

// The tile forms above, by the plan's conversion and by whether the tile is full (uniform).
template <int U, int POL, bool ZERO, bool LDS, int CVT>
__device__ __forceinline__ void move_run(const uint8_t* s, uint8_t* d, uint32_t cnt, v4u* stage) {
  const bool full = cnt == uint32_t(kReshardThreads) * U;
  if constexpr (CVT == CVT_F32_BF16 && !ZERO) {
    if (full) tile_run_f32_bf16<U, POL, true>(s, d, cnt);
    else tile_run_f32_bf16<U, POL, false>(s, d, cnt);
  } else {
    if (full) tile_run<U, POL, ZERO, LDS, CVT, true>(s, d, cnt, stage);
    else tile_run<U, POL, ZERO, LDS, CVT, false>(s, d, cnt, stage);
  }
}

template <int U, int POL, bool ZERO, bool LDS, int CVT>
__device__ __forceinline__ void move_rows(const uint8_t* s, uint8_t* d, uint32_t r0, uint32_t last, uint32_t rv,
                                          uint32_t mg, uint32_t ss, uint32_t ds, v4u* stage) {
  const bool full = last + 1 == uint32_t(kReshardThreads) * U;
  if constexpr (CVT == CVT_F32_BF16 && !ZERO) {
    if (full) tile_rows_f32_bf16<U, POL, true>(s, d, r0, last, rv, mg, ss, ds);
    else tile_rows_f32_bf16<U, POL, false>(s, d, r0, last, rv, mg, ss, ds);
  } else {
    if (full) tile_rows<U, POL, ZERO, LDS, CVT, true>(s, d, r0, last, rv, mg, ss, ds, stage);
    else tile_rows<U, POL, ZERO, LDS, CVT, false>(s, d, r0, last, rv, mg, ss, ds, stage);
  }
}

// Segments at any alignment: cnt units (any_unit_bytes destination bytes each) of rows of `run` bytes. A
// row's units sit on a grid of the destination's addresses: unit c covers the row's bytes [x, x + unit) with
// x = c * unit - (row address & gmask), cut to the row by moving the first and the last one inward. A unit
// moved inward overlaps its neighbour, and both write the same bytes there, so every access is a whole unit:
// no head or tail bytes, no read outside the row, and every other store is aligned. Units of the 128-byte
// grid also keep a tile's ends on cache lines, so that two tiles share a line only at a row's ends.
//
// ROWS: the units are numbered row-major from r0 in row 0 (at s and d), rv per row; lo and hi, the range
// of the first byte of a unit, are those of a row. Otherwise: one row's slice, lo and hi relative to s and
// d and possibly below 0.
//
// Bound by HBM. Against a tile per row slice with byte heads and tails, bodies realigned in registers and
// conversions element by element: a 12-layer decoder with odd widths (460 MB of bf16 shards, TP1 PP2 -> TP2)
// 202 -> 150 us, its fp32 -> bf16 conversion 757 -> 221 us, the 8B set into buckets of 2^28 - 2 bytes and out
// of them 12.8 -> 10.4 ms (64 GB moved).
constexpr uint32_t kAnyBias = 256;  // keeps the lanes' unsigned offsets from the base above 0

template <int CVT>
constexpr uint32_t any_src(uint32_t n) {  // source bytes behind n destination bytes
  return CVT == CVT_F32_BF16 ? n * 2 : CVT == CVT_BF16_F32 ? n / 2 : n;
}

template <int U, int POL, bool ZERO, int CVT, bool ROWS>
__device__ __forceinline__ void tile_any(const uint8_t* s, uint8_t* d, uint32_t r0, uint32_t cnt, uint32_t rv,
                                         uint32_t mg, uint32_t ss, uint32_t ds, uint32_t gmask, int32_t lo, int32_t hi) {
  constexpr uint32_t D = ZERO ? 16u : any_unit_bytes(CVT);
  constexpr int N = U * 16 / int(D), P = N > 8 ? 8 : N;  // units per lane, at most 8 of them in flight
  const uint32_t tid = threadIdx.x, a0 = uint32_t(reinterpret_cast<uintptr_t>(d));
  s = ZERO ? nullptr : s - any_src<CVT>(kAnyBias);
  d -= kAnyBias;
#pragma nounroll
  for (uint32_t b = 0; b < cnt; b += uint32_t(kReshardThreads) * P) {  // ceil(cnt / (64 P)) passes
    uint32_t to[P];
    bool live[P];
    std::conditional_t<CVT == CVT_BF16_F32 && !ZERO, v2u, v4u> r[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const uint32_t i = b + k * kReshardThreads + tid, n = r0 + umin(i, cnt - 1);
      const uint32_t q = !ROWS ? 0 : rv > 1 ? __umulhi(n, mg) : n;
      const int32_t x = int32_t((n - q * rv) * D - ((a0 + q * ds) & gmask));
      int32_t o = x < lo ? lo : x;
      o = o > hi ? hi : o;
      const uint32_t at = uint32_t(o) + kAnyBias;
      live[k] = i < cnt && x < hi + int32_t(D) && x + int32_t(D) > lo;
      to[k] = (ROWS ? q * ds : 0) + at;
      const uint32_t from = (ROWS ? q * ss : 0) + any_src<CVT>(at);
      if constexpr (ZERO) {
        r[k] = v4u{0, 0, 0, 0};
      } else if constexpr (CVT == CVT_BF16_F32) {
        r[k] = ld8_any<POL>(s, from);
      } else {
        r[k] = ld16_any<POL>(s, from);
      }
    }
    if constexpr (!ZERO) loads_done(r);
#pragma unroll
    for (int k = 0; k < P; ++k) {
      if (!live[k]) continue;
      if constexpr (CVT == CVT_F32_BF16 && !ZERO) {
        st8_any<POL>(d, to[k], to_bf16x4(r[k]));
      } else if constexpr (CVT == CVT_BF16_F32 && !ZERO) {
        st16_any<POL>(d, to[k], v4u{r[k].x << 16, r[k].x & 0xffff0000u, r[k].y << 16, r[k].y & 0xffff0000u});
      } else {
        st16_any<POL>(d, to[k], r[k]);
      }
    }
  }
}

// A whole tile of units inside one row: aligned at d, at any element of the source, nothing to cut and no lane
// masked. It is what lets such plans write through (see reshard_rule); by itself it gained under 1%.
template <int U, int POL, bool ZERO, int CVT>
__device__ __forceinline__ void tile_inner(const uint8_t* s, uint8_t* d) {
  constexpr uint32_t D = ZERO ? 16u : any_unit_bytes(CVT);
  constexpr int N = U * 16 / int(D), P = N > 8 ? 8 : N;
  const uint32_t tid = threadIdx.x;
#pragma unroll
  for (int b = 0; b < N; b += P) {
    v4u r[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const uint32_t from = any_src<CVT>(((b + k) * kReshardThreads + tid) * D);
      if constexpr (ZERO) {
        r[k] = v4u{0, 0, 0, 0};
      } else if constexpr (CVT == CVT_BF16_F32) {
        const v2u h = ld8_any<POL>(s, from);
        r[k].x = h.x;
        r[k].y = h.y;
      } else {
        r[k] = ld16_any<POL>(s, from);
      }
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const uint32_t to = ((b + k) * kReshardThreads + tid) * D;
      if constexpr (CVT == CVT_F32_BF16 && !ZERO) {
        st8<POL>(d, to, to_bf16x4(r[k]));
      } else if constexpr (CVT == CVT_BF16_F32 && !ZERO) {
        st16<POL>(d, to, v4u{r[k].x << 16, r[k].x & 0xffff0000u, r[k].y << 16, r[k].y & 0xffff0000u});
      } else {
        st16<POL>(d, to, r[k]);
      }
    }
  }
}

// Rows shorter than a unit (narrow column slices, the ends of bucket-cut rows): element by element, one per
// lane and step, in row-major order.
template <int U, bool ZERO, int CVT>
__device__ void tile_elems(const DevSeg& g, uint64_t lt, const uint8_t* sb, uint8_t* db) {
  typedef const __attribute__((address_space(1))) uint32_t* g32;
  typedef const __attribute__((address_space(1))) uint16_t* g16;
  constexpr uint32_t ES = CVT == CVT_BF16_F32 && !ZERO ? 4 : 2;
  const uint64_t per = g.run / ES, total = g.rows * per;
  for (uint32_t u = 0; u < U; ++u) {
    const uint64_t e = lt * (uint64_t(kReshardThreads) * U) + u * kReshardThreads + threadIdx.x;
    if (e >= total) return;
    const uint64_t row = e / per, o = (e - row * per) * ES;
    gu8* d = (gu8*)db + g.dst_off + row * g.dst_stride + o;
    const gu8* s = (const gu8*)sb + g.src_off + row * g.src_stride;
    if constexpr (ZERO) *(__attribute__((address_space(1))) uint16_t*)d = 0;
    else if constexpr (CVT == CVT_F32_BF16) *(__attribute__((address_space(1))) uint16_t*)d = uint16_t(bf16_rne(*(g32)(s + o * 2)));
    else if constexpr (CVT == CVT_BF16_F32) *(__attribute__((address_space(1))) uint32_t*)d = uint32_t(*(g16)(s + o / 2)) << 16;
    else *(__attribute__((address_space(1))) uint16_t*)d = *(g16)(s + o);
  }
}

template <int U, int POL, bool ZERO, bool LDS, int CVT>
__device__ __forceinline__ void run_tile(const DevSeg& g, uint64_t lt, const uint8_t* sb, uint8_t* db, v4u* stage) {
  constexpr uint64_t TV = uint64_t(kReshardThreads) * U;
  constexpr uint64_t SV = kSrcVecBytes<CVT>;
  const uint32_t mode = g.mode & SEG_MODE_MASK;
  if (mode == SEG_VEC_1D) {
    const uint64_t nv = g.run / 16, v0 = lt * TV;
    const uint32_t cnt = uint32_t(nv - v0 < TV ? nv - v0 : TV);
    move_run<U, POL, ZERO, LDS, CVT>(ZERO ? nullptr : sb + g.src_off + v0 * SV, db + g.dst_off + v0 * 16, cnt, stage);
  } else if (mode == SEG_VEC_FLAT || mode == SEG_VEC_ROWS) {
    // FLAT: vectors [lt * TV, lt * TV + TV) of the rows' row-major order, starting in row row0 at
    // column r0. ROWS: `param` whole rows per tile.
    uint64_t row0;
    uint32_t r0, last;
    if (mode == SEG_VEC_FLAT) {
      const uint32_t n0 = uint32_t(lt) * uint32_t(TV);  // below param = rows * rv < 2^32
      const uint32_t q0 = g.rv > 1 ? __umulhi(n0, g.magic) : n0;
      row0 = q0;
      r0 = n0 - q0 * g.rv;
      last = umin(g.param - n0, uint32_t(TV)) - 1;
    } else {
      row0 = lt * g.param;
      r0 = 0;
      last = uint32_t(g.rows - row0 < g.param ? g.rows - row0 : g.param) * g.rv - 1;
    }
    const uint8_t* s = ZERO ? nullptr : sb + g.src_off + row0 * g.src_stride;
    uint8_t* d = db + g.dst_off + row0 * g.dst_stride;
    const uint32_t ss = uint32_t(g.src_stride), ds = uint32_t(g.dst_stride);
    move_rows<U, POL, ZERO, LDS, CVT>(s, d, r0, last, g.rv, g.magic, ss, ds, stage);
  } else if (mode == SEG_VEC_ROWCHUNK) {
    const uint64_t row = lt / g.param, ch = lt - row * g.param;
    const uint64_t nv = g.run / 16, v0 = ch * TV;
    const uint32_t cnt = uint32_t(nv - v0 < TV ? nv - v0 : TV);
    const uint8_t* s = ZERO ? nullptr : sb + g.src_off + row * g.src_stride + v0 * SV;
    uint8_t* d = db + g.dst_off + row * g.dst_stride + v0 * 16;
    move_run<U, POL, ZERO, LDS, CVT>(s, d, cnt, stage);
  } else if (mode == SEG_ANY_FLAT) {
    constexpr uint32_t D = ZERO ? 16u : any_unit_bytes(CVT), TU = uint32_t(TV) * 16 / D;  // units per tile
    const uint32_t n0 = uint32_t(lt) * TU, q0 = g.rv > 1 ? __umulhi(n0, g.magic) : n0, r0 = n0 - q0 * g.rv;
    const uint32_t gmask = g.mode >> SEG_GRID_SHIFT;
    const uint8_t* s = ZERO ? nullptr : sb + g.src_off + uint64_t(q0) * g.src_stride;
    uint8_t* d = db + g.dst_off + uint64_t(q0) * g.dst_stride;
    // A row's first unit on the grid is among its first 128 bytes of units, and its last among the last 256:
    // a row has less than 256 bytes more of units than of data.
    if (r0 * D >= 128 && (r0 + TU) * D + 256 <= g.rv * D) {
      const uint32_t at = r0 * D - (uint32_t(reinterpret_cast<uintptr_t>(d)) & gmask);
      tile_inner<U, POL, ZERO, CVT>(s + any_src<CVT>(at), d + at);
    } else {
      tile_any<U, POL, ZERO, CVT, true>(s, d, r0, umin(g.param - n0, TU), g.rv, g.magic, uint32_t(g.src_stride),
                                        uint32_t(g.dst_stride), gmask, 0, int32_t(g.run) - int32_t(D));
    }
  } else if (mode == SEG_ANY_CHUNK) {
    // Slice ch of a row is its bytes [ch * TB - m, (ch + 1) * TB - m), cut to the row, with m the phase of the
    // row's address on the grid; the last slice also takes what is left (up to gmask bytes).
    constexpr uint32_t D = ZERO ? 16u : any_unit_bytes(CVT);
    constexpr int32_t TB = int32_t(TV) * 16;
    const uint32_t row = g.rows == 1 ? 0 : uint32_t(lt) / g.param, ch = uint32_t(lt) - row * g.param;
    const uint64_t b0 = uint64_t(ch) * uint32_t(TB);
    const uint8_t* s = ZERO ? nullptr : sb + g.src_off + row * g.src_stride + b0 / 16 * SV;
    uint8_t* d = db + g.dst_off + row * g.dst_stride + b0;
    const uint32_t gmask = g.mode >> SEG_GRID_SHIFT;
    const int32_t m = int32_t(uint32_t(reinterpret_cast<uintptr_t>(d)) & gmask);
    if (ch != 0 && ch + 1 != g.param) {
      tile_inner<U, POL, ZERO, CVT>(s - any_src<CVT>(uint32_t(m)), d - m);
    } else {
      const int32_t end = ch + 1 == g.param ? int32_t(g.run - b0) : TB - m;
      tile_any<U, POL, ZERO, CVT, false>(s, d, 0, (uint32_t(end + m) + D - 1) / D, 0, 0, 0, 0, gmask, ch ? -m : 0,
                                         end - int32_t(D));
    }
  } else {
    tile_elems<U, ZERO, CVT>(g, lt, sb, db);
  }
}

// One workgroup per tile. The dispatcher deals workgroups to the XCDs round-robin; with XCD remapping, XCD x
// takes blocks x, x + 8, ... of kReshardBlock consecutive tiles (1 MB at 4 KB tiles), so each XCD's L2 sees
// whole blocks and the eight of them work through one front of the map; what is left after the last whole
// round of blocks, or all of a map that reshard_rule gives no blocks, goes to the XCDs in contiguous eighths. On the same buffers, 1B TP4 -> TP2 / the same in
// fp32, three groups / 8B TP2 PP2 -> TP4: 885 / 5356 / 4822 us against 901 / 5398 / 4799 with contiguous
// eighths of the whole map; blocks of 512 tiles 887 / 5372 / 4812, of 1024 891 / 5370 / 4816.
//
// The map holds the copy segments' tiles, then the zero-fill segments' (padded vocabulary rows); both run in
// one launch: a launch of its own took the zero fill 4 to 5 us, whatever its size.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t w, uint32_t per, uint32_t whole) {  // per: an eighth of the
  const uint32_t x = w % kXcds, j = w / kXcds;                                              // grid; whole: in blocks
  if (j < whole) return ((j / kReshardBlock) * kXcds + x) * kReshardBlock + j % kReshardBlock;
  return whole * kXcds + x * (per - whole) + (j - whole);
}

template <int U, int POL, bool LDS, bool XCD, int CVT>
__global__ __launch_bounds__(kReshardThreads, EMU_RESHARD_WAVES_PER_EU) void k_reshard(const uint32_t* __restrict__ tilemap,
                                                                             uint32_t tile_base, uint32_t per,
                                                                             uint32_t whole,
                                                                             const DevSeg* __restrict__ segs,
                                                                             const uint64_t* __restrict__ dst_ptrs,
                                                                             const uint64_t* __restrict__ src_ptrs,
                                                                             uint32_t dst_n, uint32_t src_n) {
  extern __shared__ v4u stage[];
  // Each section of the map is padded with kNoSeg to a multiple of the XCD count, so no bounds check
  // precedes the map load. The source pointer's load issues together with the destination pointer's, right
  // after the descriptor, also where a zero fill will not use it (entry 0 then): the chain before the first
  // data load is map entry, descriptor, pointers. The arguments are in registers when a wave starts (the
  // build asks for them to be preloaded).
  const uint32_t tile = tile_base + (XCD ? xcd_tile(blockIdx.x, per, whole) : blockIdx.x);
  const uint32_t si = tilemap[tile];
  if (si == kNoSeg) return;
  const DevSeg g = segs[si];
  // grid row y runs tensor group y: its pointer tables follow the earlier groups' back to back
  uint8_t* db = reinterpret_cast<uint8_t*>(dst_ptrs[uint64_t(blockIdx.y) * dst_n + g.dst_idx]);
  const uint8_t* sb =
      reinterpret_cast<const uint8_t*>(src_ptrs[uint64_t(blockIdx.y) * src_n + (g.src_idx < 0 ? 0 : g.src_idx)]);
  const uint32_t lt = tile - uint32_t(g.tile0);
  if (g.mode & SEG_ZERO) run_tile<U, POL, true, LDS, CVT_NONE>(g, lt, nullptr, db, stage);
  else run_tile<U, POL, false, LDS, CVT>(g, lt, sb, db, stage);
}

// ------------------------------------------------------------------------------------------------
// bucket pack / unpack kernel
// ------------------------------------------------------------------------------------------------
// Work unit: a chunk of kChunkBytes of one rank's stream. When a workgroup reaches a new rank it
// computes, in LDS, the exclusive prefix sum of that rank's ragged tensor sizes with a wave64 scan
// (wave 0), and the index of the rank's first bucket, sum over earlier ranks of ceil(bytes / B),
// with a wave64 reduction (wave 1). A chunk is then cut at tensor and bucket boundaries into pieces,
// each copied by the whole workgroup.

__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v, uint32_t lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(v, d, 64);
    if (lane >= uint32_t(d)) v += y;
  }
  return v;
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

template <bool UNPACK, int POL, int U>
__global__ __launch_bounds__(kThreads, EMU_BUCKET_WAVES_PER_EU) void k_buckets(const uint64_t* __restrict__ sizes,
                                                      const uint32_t* __restrict__ rank_first,
                                                      const uint64_t* __restrict__ rank_bytes,
                                                      const uint64_t* __restrict__ chunk_first, int32_t nranks,
                                                      uint64_t B, const uint64_t* __restrict__ tensor_ptrs,
                                                      const uint64_t* __restrict__ bucket_ptrs) {
  __shared__ uint64_t offs[kMaxRankTensors + 1];
  __shared__ uint64_t s_bucket0;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t nchunks = chunk_first[nranks];
  // XCD-aware chunk order: with a grid that is a multiple of the XCD count, the workgroups of XCD x
  // (x, x+8, ...) stride through the contiguous eighth [x*N/8, (x+1)*N/8) of the chunks.
  uint64_t c_begin = blockIdx.x, c_end = nchunks, c_step = gridDim.x;
  if (gridDim.x % kXcds == 0) {
    const uint32_t x = blockIdx.x % kXcds;
    c_begin = nchunks * x / kXcds + blockIdx.x / kXcds;
    c_end = nchunks * (x + 1) / kXcds;
    c_step = gridDim.x / kXcds;
  }
  int32_t r = 0, cur = -1;
  uint32_t t0 = 0, nt = 0, ti = 0;
  uint64_t bucket0 = 0;
  for (uint64_t c = c_begin; c < c_end; c += c_step) {
    while (chunk_first[r + 1] <= c) ++r;
    if (r != cur) {
      __syncthreads();  // previous rank's offsets no longer read
      t0 = rank_first[r];
      nt = rank_first[r + 1] - t0;
      if (wave == 0) {
        uint64_t carry = 0;
        for (uint32_t base = 0; base < nt; base += 64) {
          const uint32_t i = base + lane;
          const uint64_t incl = wave_incl_scan(i < nt ? sizes[t0 + i] : 0, lane);
          if (i < nt) offs[i + 1] = carry + incl;
          carry += __shfl(incl, 63, 64);
        }
        if (lane == 0) offs[0] = 0;
      } else if (wave == 1) {
        uint64_t acc = 0;
        for (int32_t q = lane; q < r; q += 64) acc += (rank_bytes[q] + B - 1) / B;
        acc = wave_sum(acc);
        if (lane == 0) s_bucket0 = acc;
      }
      __syncthreads();
      cur = r;
      ti = 0;
      bucket0 = uniform64(s_bucket0);
    }
    const uint64_t S = uniform64(offs[nt]);
    const uint64_t start = (c - chunk_first[r]) * kChunkBytes;
    const uint64_t end = start + kChunkBytes < S ? start + kChunkBytes : S;
    // tensor holding `start`: chunks of one workgroup move forward through the rank, so walk on from
    // the previous chunk's tensor when it is close, else binary-search the offsets
    if (offs[ti] > start || (ti + 8 < nt && offs[ti + 8] <= start)) {
      uint32_t lo = 0, hi = nt;
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (offs[mid] <= start) lo = mid; else hi = mid;
      }
      ti = lo;
    }
    ti = __builtin_amdgcn_readfirstlane(ti);
    uint64_t k = start / B;            // bucket of `start`; advanced incrementally below
    uint64_t kend = (k + 1) * B;
    uint64_t pos = start;
    while (pos < end) {
      while (uniform64(offs[ti + 1]) <= pos) ti = __builtin_amdgcn_readfirstlane(ti + 1);  // skips empty tensors
      const uint64_t toff = uniform64(offs[ti]), tend = uniform64(offs[ti + 1]);
      uint64_t pend = end < tend ? end : tend;
      if (kend < pend) pend = kend;
      uint8_t* tp = reinterpret_cast<uint8_t*>(tensor_ptrs[t0 + ti]) + (pos - toff);
      uint8_t* bp = reinterpret_cast<uint8_t*>(bucket_ptrs[bucket0 + k]) + (pos - k * B);
      const uint32_t n = uint32_t(pend - pos);
      if constexpr (UNPACK) wg_copy<kThreads, U, POL>(bp, tp, n, uint32_t(pos - toff) & 15u);
      else wg_copy<kThreads, U, POL>(tp, bp, n, uint32_t(pos - k * B) & 15u);
      pos = pend;
      if (pos == kend) {
        ++k;
        kend += B;
      }
    }
  }
}

// Tile-per-workgroup variant: one workgroup per 4 KB chunk (kTileChunkBytes) of one rank's stream, in
// block-cyclic XCD order. The upload-time map gives the chunk's rank and the global index of the tensor
// holding its first byte, so the tensor's stream range and pointer load in parallel with the rank's
// record; the map is padded to the grid, so no bounds check precedes it. The rank's first bucket, the
// sum over earlier ranks of ceil(bytes / B), comes from the host in a kernel argument for the first
// kArgRanks ranks, else from a wave64 reduction. The chunk is then cut at tensor and bucket boundaries.
//
// Chunk ends sit on the destination's 4 KB grid. For aligned buckets and tensors that is the stream's
// grid. When it is not (REALIGN: pack into buckets whose size is not a multiple of 4 KB, unpack into tensors
// whose stream offsets are not), both ends of every chunk move down to the destination's grid, by the same
// rule on either side of each cut, so consecutive chunks still tile the stream. Every destination cache
// line is then written by one workgroup; cut on the stream's grid, every chunk end would split a line
// between two workgroups, which costs partial-line writes to HBM.
constexpr int kArgRanks = 128;
// Chunks per block of the bucket kernel's XCD order (64 x 4 KB = 256 KB). Contiguous eighths per XCD put the
// eight XCD streams exactly one eighth of the streams apart; on a rank set laid out
// in one allocation that ran pack and unpack at 75-80% of HBM peak against 82% in per-rank buffers. Blocks of
// 256 KB ran both layouts at 82%; 64 KB and 128 KB blocks lost 5-12 points, 512 KB to 2 MB blocks 0.3-1.
constexpr uint32_t kBucketBlock = 64;
struct BucketBases {
  uint64_t first[kArgRanks];  // first bucket of each rank, for ranks below kArgRanks
};

// floor(x / B) with recip = floor((2^64 - 1) / B): the product's high half is at most two short.
__device__ __forceinline__ uint64_t div_by(uint64_t x, uint64_t B, uint64_t recip) {
  uint64_t k = __umul64hi(x, recip);
  while (x - k * B >= B) ++k;
  return k;
}

template <bool UNPACK, int POL, int U, bool REALIGN>
__global__ __launch_bounds__(kBucketTileThreads, EMU_RESHARD_WAVES_PER_EU) void k_buckets_tile(
    const uint32_t* __restrict__ tile_map, uint32_t n_map, const uint64_t* __restrict__ rank_info,
    const uint64_t* __restrict__ stream_off, const uint64_t* __restrict__ tensor_ptrs,
    const uint64_t* __restrict__ bucket_ptrs, uint64_t B, uint64_t recip, const uint64_t* __restrict__ rank_bytes,
    BucketBases bases) {
  // Block-cyclic order: the dispatcher deals workgroups to the XCDs round-robin, and XCD x takes blocks
  // x, x + 8, ... of kBucketBlock consecutive chunks, so the eight XCDs stream through neighbouring
  // 256 KB blocks of one front. The map's tail past the last whole round of blocks keeps plain order
  // (the mapping stays a bijection on the padded map). See kBucketBlock.
  constexpr uint32_t kTensor = (1u << kMapTensorBits) - 1;
  const uint32_t w = blockIdx.x, full = n_map / (kXcds * kBucketBlock) * (kXcds * kBucketBlock);
  const uint32_t j = w / kXcds;
  const uint32_t c = w < full ? ((j / kBucketBlock) * kXcds + w % kXcds) * kBucketBlock + j % kBucketBlock : w;
  const uint32_t m = tile_map[c];
  const uint32_t next = UNPACK && REALIGN ? tile_map[umin(c + 1, n_map - 1)] & kTensor : 0;  // the next chunk's tensor
  if (m == kNoSeg) return;
  const uint32_t r = m >> kMapTensorBits;
  uint32_t g = m & kTensor;
  const uint64_t c0 = rank_info[4 * r], S = rank_info[4 * r + 1];
  const uint32_t gend = uint32_t(rank_info[4 * r + 2]);
  // Tensor g's stream range and pointer. A rank's last tensor has no end among its rank's offsets: S stands
  // in, and what is loaded behind the last offset of all (the rank records) is not used.
  uint64_t toff = stream_off[g], tnext = stream_off[g + 1];
  uint64_t tptr = tensor_ptrs[g];
  uint64_t bucket0;
  if (r < uint32_t(kArgRanks)) {
    bucket0 = bases.first[r];
  } else {
    const uint32_t lane = threadIdx.x & 63;
    uint64_t acc = 0;
    for (uint32_t q = lane; q < r; q += 64) acc += div_by(rank_bytes[q] + B - 1, B, recip);
    bucket0 = uniform64(wave_sum(acc));
  }
  uint64_t start = (c - c0) * kTileChunkBytes;
  uint64_t end = start + kTileChunkBytes < S ? start + kTileChunkBytes : S;
  uint64_t k = div_by(start, B, recip);
  if constexpr (REALIGN) {
    // pack: bucket k's grid starts at stream byte k*B; unpack: a tensor's grid starts at its stream
    // offset (the tensor holding `end` is the next chunk's map entry). A start never leaves its bucket
    // (pack) or tensor (unpack); it may move back into earlier tensors (pack) or an earlier bucket
    // (unpack). Chunks stay non-empty and below 2 * kTileChunkBytes.
    constexpr uint64_t kGrid = kTileChunkBytes - 1;
    if constexpr (UNPACK) {
      start -= (start - toff) & kGrid;
      if (end < S) end -= (end - stream_off[next]) & kGrid;
      k = div_by(start, B, recip);
    } else {
      start -= (start - k * B) & kGrid;
      if (end < S) end -= (end - div_by(end, B, recip) * B) & kGrid;
      if (toff > start) {
        while (stream_off[g] > start) --g;
        toff = stream_off[g];
        tnext = stream_off[g + 1];
        tptr = tensor_ptrs[g];
      }
    }
  }
  uint64_t kend = (k + 1) * B;
  uint64_t pos = start;
  while (pos < end) {
    const uint64_t tend = g + 1 < gend ? tnext : S;
    if (tend <= pos) {  // the chunk moves on into the next tensor (or past an empty one)
      ++g;
      toff = tnext;
      tnext = stream_off[g + 1];
      tptr = tensor_ptrs[g];
      continue;
    }
    uint64_t pend = end < tend ? end : tend;
    if (kend < pend) pend = kend;
    uint8_t* tp = reinterpret_cast<uint8_t*>(tptr) + (pos - toff);
    uint8_t* bp = reinterpret_cast<uint8_t*>(bucket_ptrs[bucket0 + k]) + (pos - k * B);
    const uint32_t n = uint32_t(pend - pos);
    if constexpr (UNPACK) wg_copy<kBucketTileThreads, U, POL>(bp, tp, n, uint32_t(pos - toff) & 15u);
    else wg_copy<kBucketTileThreads, U, POL>(tp, bp, n, uint32_t(pos - k * B) & 15u);
    pos = pend;
    if (pos == kend) {
      ++k;
      kend += B;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// upload-time tables
// ------------------------------------------------------------------------------------------------
// emu_plan_upload copies the segments with their tile counts and each side's host tables (tensor sizes,
// each rank's tensor range and stream length), and derives the rest on the device.
//
// k_tile_map: workgroup x < n_seg writes segment x's index into its tiles' map entries, from the
// segment's first map index on (workgroups y = 0, 1, ... stride through a long segment); workgroup n_seg
// fills the padding after each section (copy tiles, zero-fill tiles) with kNoSeg.
__global__ __launch_bounds__(256) void k_tile_map(const DevSeg* __restrict__ segs,
                                                  const uint32_t* __restrict__ seg_tiles, uint32_t n_seg,
                                                  uint32_t* __restrict__ map, uint64_t copy_end, uint64_t zero0,
                                                  uint64_t zero_end, uint64_t n_map) {
  const uint32_t x = blockIdx.x;
  if (x == n_seg) {
    if (blockIdx.y != 0) return;
    for (uint64_t j = copy_end + threadIdx.x; j < zero0; j += blockDim.x) map[j] = kNoSeg;
    for (uint64_t j = zero_end + threadIdx.x; j < n_map; j += blockDim.x) map[j] = kNoSeg;
    return;
  }
  const uint64_t t0 = segs[x].tile0;
  const uint32_t n = seg_tiles[x];
  for (uint64_t j = uint64_t(blockIdx.y) * blockDim.x + threadIdx.x; j < n; j += uint64_t(gridDim.y) * blockDim.x)
    map[t0 + j] = x;
}

// k_stream_tables, one wave64 per rank: the
// exclusive prefix sum of the rank's tensor sizes (each tensor's stream offset), and the rank's record
// {first 4 KB chunk, stream bytes, end of its tensor range, 0}, whose first chunk is the sum over earlier
// ranks of ceil(bytes / 4 KB).
__global__ __launch_bounds__(64) void k_stream_tables(const uint64_t* __restrict__ sizes,
                                                      const uint32_t* __restrict__ rank_first,
                                                      const uint64_t* __restrict__ rank_bytes,
                                                      uint64_t* __restrict__ stream_off,
                                                      uint64_t* __restrict__ rank_info) {
  const uint32_t r = blockIdx.x, lane = threadIdx.x;
  const uint32_t t0 = rank_first[r], t1 = rank_first[r + 1];
  uint64_t carry = 0;
  for (uint32_t base = t0; base < t1; base += 64) {
    const uint32_t i = base + lane;
    const uint64_t v = i < t1 ? sizes[i] : 0;
    const uint64_t incl = wave_incl_scan(v, lane);
    if (i < t1) stream_off[i] = carry + incl - v;
    carry += __shfl(incl, 63, 64);
  }
  uint64_t acc = 0;
  for (uint32_t q = lane; q < r; q += 64) acc += (rank_bytes[q] + kTileChunkBytes - 1) / kTileChunkBytes;
  acc = wave_sum(acc);
  if (lane == 0) {
    rank_info[4 * r + 0] = acc;
    rank_info[4 * r + 1] = rank_bytes[r];
    rank_info[4 * r + 2] = t1;
    rank_info[4 * r + 3] = 0;
  }
}

// The chunk map, after k_stream_tables: workgroup g < n_tensors gives every chunk of g's rank whose first
// byte lies in tensor g the entry rank << 20 | g (chunk j of a rank starts in the last tensor whose stream
// offset is <= j * 4 KB: chunks ceil(offset_g / 4 KB) up to ceil(offset_g+1 / 4 KB), or to the rank's
// chunk count for its last tensor), and workgroup n_tensors fills the map's padding after the last
// rank's chunks with kNoSeg.
__global__ __launch_bounds__(256) void k_chunk_map(const uint32_t* __restrict__ rank_first,
                                                   const uint64_t* __restrict__ rank_bytes, uint32_t nranks,
                                                   uint32_t n_tensors, const uint64_t* __restrict__ stream_off,
                                                   const uint64_t* __restrict__ rank_info,
                                                   uint32_t* __restrict__ map, uint64_t n_map) {
  constexpr uint64_t C = kTileChunkBytes;
  const uint32_t g = blockIdx.x;
  uint64_t first = 0, j0, j1;
  uint32_t v = kNoSeg;
  if (g == n_tensors) {
    j0 = rank_info[4 * (nranks - 1)] + (rank_bytes[nranks - 1] + C - 1) / C;
    j1 = n_map;
  } else {
    uint32_t lo = 0, hi = nranks;  // the rank r with rank_first[r] <= g < rank_first[r + 1]
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (rank_first[mid] <= g) lo = mid; else hi = mid;
    }
    const uint32_t t1 = rank_first[lo + 1];
    first = rank_info[4 * lo];
    j0 = (stream_off[g] + C - 1) / C;
    j1 = g + 1 < t1 ? (stream_off[g + 1] + C - 1) / C : (rank_bytes[lo] + C - 1) / C;
    v = (lo << kMapTensorBits) | g;
  }
  for (uint64_t j = j0 + threadIdx.x; j < j1; j += blockDim.x) map[first + j] = v;
}

// ------------------------------------------------------------------------------------------------
// launch helpers
// ------------------------------------------------------------------------------------------------

// A device attribute of the current device, cached per device (0 when it cannot be read).
static int device_attr(hipDeviceAttribute_t attr, int slot) {
  static std::atomic<int> cache[3][64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  const bool cached = dev >= 0 && dev < 64;
  if (cached) {
    const int v = cache[slot][dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
  }
  int v = 0;
  if (hipDeviceGetAttribute(&v, attr, dev) != hipSuccess || v <= 0) return 0;
  if (cached) cache[slot][dev].store(v, std::memory_order_relaxed);
  return v;
}

static int device_cus() {
  const int v = device_attr(hipDeviceAttributeMultiprocessorCount, 0);
  return v > 0 ? v : -1;
}

// Dynamic LDS for a tile kernel that needs `need` bytes. A residency cap of `cap` workgroups per CU is
// enforced by reserving the CU's LDS divided by cap, rounded down to whole KB; the kernels never touch the
// reserved bytes. The CU's LDS is allocated in two halves and a workgroup's block lies in one half, so the
// resident count is 2 * floor(cap / 2) for cap >= 2 (1 keeps one).
static size_t occupancy_lds(size_t need, int cap) {
  if (cap == 0) return need;
  const int per_cu = device_attr(hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, 1);
  const int per_wg = device_attr(hipDeviceAttributeMaxSharedMemoryPerBlock, 2);
  if (per_cu <= 0 || per_wg <= 0) return need;
  size_t r = (size_t(per_cu) / size_t(cap)) & ~size_t(1023);
  if (r > size_t(per_wg)) r = size_t(per_wg);
  return r > need ? r : need;
}

// Kernel launches report through the runtime's per-thread last-error state. An error some earlier
// runtime call left there belongs to that call, which has already returned it: it is dropped before the
// library launches, so that hip_check afterwards sees only the library's own launches.
static void drop_pending_error() { (void)hipGetLastError(); }

static int hip_check(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(EMU_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
  return EMU_OK;
}

// Pointer tables of one reshard launch: `groups` source and destination tables back to back, each group
// src_n source and dst_n destination entries (one group for emu_reshard).
struct Tables {
  const uint64_t* sp;
  const uint64_t* dp;
  uint32_t groups, src_n, dst_n;
};

// Launches k_reshard over the whole map (n_map entries, a multiple of kXcds) for every group (grid row y =
// group y).
struct ReshardLaunch {
  const DevSeg* segs;
  const uint32_t* tm;
  uint64_t n_map;
  int cap;
  bool blocks;
  Tables tb;
  hipStream_t st;
};

template <int U, int POL, bool LDS, bool XCD, int CVT>
static void launch_reshard(const ReshardLaunch& l) {
  constexpr uint64_t kTile = uint64_t(kReshardThreads) * U * 16;
  const size_t lds = occupancy_lds(LDS ? size_t(kTile) : 0, l.cap);
  // a multiple of kXcds whose work-items (64 per workgroup) stay below 2^32 in the grid's x dimension
  constexpr uint64_t kMaxGrid = (1ull << 26) - kXcds;
  for (uint64_t done = 0; done < l.n_map; done += kMaxGrid) {
    const uint32_t grid = uint32_t(l.n_map - done < kMaxGrid ? l.n_map - done : kMaxGrid), per = grid / kXcds;
    hipLaunchKernelGGL((k_reshard<U, POL, LDS, XCD, CVT>), dim3(grid, l.tb.groups), dim3(kReshardThreads), lds, l.st,
                       l.tm, uint32_t(done), per, l.blocks ? per / kReshardBlock * kReshardBlock : 0u, l.segs, l.tb.dp, l.tb.sp, l.tb.dst_n, l.tb.src_n);
  }
}

// For every combination of the launch options (LDS staging and XCD order; converting plans: no LDS staging).
template <int U, int POL, int CVT>
static void launch_options(const ReshardLaunch& l) {
  const bool xcd = option(EMU_OPT_XCD_REMAP) != 0;
  if constexpr (CVT == CVT_NONE) {
    if (option(EMU_OPT_LDS_STAGING) != 0)
      return xcd ? launch_reshard<U, POL, true, true, CVT>(l) : launch_reshard<U, POL, true, false, CVT>(l);
  }
  xcd ? launch_reshard<U, POL, false, true, CVT>(l) : launch_reshard<U, POL, false, false, CVT>(l);
}

template <int U, int CVT>
static void launch_policy(int policy, const ReshardLaunch& l) {
  if (policy == POL_PLAIN) launch_options<U, POL_PLAIN, CVT>(l);
  else if (policy == POL_THROUGH) launch_options<U, POL_THROUGH, CVT>(l);
  else launch_options<U, POL_NT, CVT>(l);
}

template <int U>
static void launch_convert(int cvt, int policy, const ReshardLaunch& l) {
  switch (cvt) {
    case CVT_F32_BF16: launch_policy<U, CVT_F32_BF16>(policy, l); break;
    case CVT_BF16_F32: launch_policy<U, CVT_BF16_F32>(policy, l); break;
    default: launch_policy<U, CVT_NONE>(policy, l); break;
  }
}

static bool misaligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

static int bucket_call(emu_plan_t plan, const void* ws, int32_t side, uint64_t B, const uint64_t* tptr,
                       const uint64_t* bptr, void* stream, bool unpack) {
  clear_error();
  const Plan* P = reinterpret_cast<const Plan*>(plan);
  if (!plan_live(P)) return fail(EMU_ERR_HANDLE, "not a live plan");
  if (!ws || !tptr || !bptr) return fail(EMU_ERR_NULL, "NULL workspace or pointer table");
  if (side != 0 && side != 1) return fail(EMU_ERR_RANGE, "side must be 0 or 1");
  if (misaligned(ws, kWsAlign)) return fail(EMU_ERR_WORKSPACE, "workspace not %llu-byte aligned", (unsigned long long)kWsAlign);
  if (misaligned(tptr, 8) || misaligned(bptr, 8)) return fail(EMU_ERR_ALIGN, "pointer tables must be 8-byte aligned");
  const SideInfo& s = P->side[side];
  const uint64_t es = s.lay.dtype == EMU_BF16 ? 2 : 4;
  if (B == 0 || B % es) return fail(EMU_ERR_BUCKET, "bucket size %llu is not a positive multiple of %llu",
                                    (unsigned long long)B, (unsigned long long)es);
  for (int r = 0; r < s.nranks; ++r)
    if (s.rank_first[r + 1] - s.rank_first[r] > uint32_t(kMaxRankTensors))
      return fail(EMU_ERR_UNSUPPORTED, "rank %d has more than %d tensors on this side", r, kMaxRankTensors);
  const uint64_t nchunks = s.chunk_first[s.nranks];
  if (nchunks == 0) return EMU_OK;
  if (!ws_current(ws, P))
    return fail(EMU_ERR_WORKSPACE, "workspace %p holds no upload of this plan (fill it with emu_plan_upload)", ws);
  const int cus = device_cus();
  if (cus <= 0) return fail(EMU_ERR_HIP, "cannot query the current device");
  const uint64_t want = uint64_t(cus) * uint64_t(option(EMU_OPT_BUCKET_WG_PER_CU));
  uint64_t grid = nchunks < want ? nchunks : want;
  if (grid > kXcds) grid -= grid % kXcds;  // keep the XCD-aware chunk order available
  const uint8_t* w = static_cast<const uint8_t*>(ws);
  const SideTables& t = P->ws.side[side];
  const uint64_t* sizes = reinterpret_cast<const uint64_t*>(w + t.off_sizes);
  const uint32_t* rf = reinterpret_cast<const uint32_t*>(w + t.off_rank_first);
  const uint64_t* rb = reinterpret_cast<const uint64_t*>(w + t.off_rank_bytes);
  const uint64_t* cf = reinterpret_cast<const uint64_t*>(w + t.off_chunk_first);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool ntm = option(EMU_OPT_NONTEMPORAL) != 0;
  if (option(EMU_OPT_BUCKET_TILES) != 0 && t.n_tiles > 0) {
    const uint64_t* so = reinterpret_cast<const uint64_t*>(w + t.off_stream);
    const uint64_t* ri = reinterpret_cast<const uint64_t*>(w + t.off_rank_info);
    const uint32_t* tm = reinterpret_cast<const uint32_t*>(w + t.off_tile_map);
    BucketBases bases;
    uint64_t acc = 0;
    for (int r = 0; r < s.nranks && r < kArgRanks; ++r) {
      bases.first[r] = acc;
      acc += (s.rank_bytes[r] + B - 1) / B;
    }
    const bool realign = chunks_realign(s, B, unpack);
    const LaunchRule rule = bucket_rule(s, B, unpack);
    const dim3 g(uint32_t(t.n_tiles));  // padded to a multiple of kXcds
    const size_t lds = occupancy_lds(0, rule.cap);
    const uint64_t recip = ~0ull / B;
    drop_pending_error();
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, g, dim3(kBucketTileThreads), lds, st, tm, uint32_t(t.n_tiles), ri, so, tptr, bptr, B,
                         recip, rb, bases);
    };
    auto by_policy = [&](auto unpacks, auto realigns) {
      constexpr int U = kBucketTileVecs;
      constexpr bool kUnpack = decltype(unpacks)::value, kRealign = decltype(realigns)::value;
      if (rule.policy == POL_THROUGH) launch(k_buckets_tile<kUnpack, POL_THROUGH, U, kRealign>);
      else if (rule.policy == POL_NT) launch(k_buckets_tile<kUnpack, POL_NT, U, kRealign>);
      else launch(k_buckets_tile<kUnpack, POL_PLAIN, U, kRealign>);
    };
    if (unpack) realign ? by_policy(std::true_type(), std::true_type()) : by_policy(std::true_type(), std::false_type());
    else realign ? by_policy(std::false_type(), std::true_type()) : by_policy(std::false_type(), std::false_type());
    return hip_check(unpack ? "emu_unpack_buckets launch" : "emu_pack_buckets launch");
  }
  drop_pending_error();
  if (unpack) {
    if (ntm) hipLaunchKernelGGL((k_buckets<true, POL_NT, kBucketUnroll>), dim3(uint32_t(grid)), dim3(kThreads), 0, st, sizes, rf, rb, cf, s.nranks, B, tptr, bptr);
    else hipLaunchKernelGGL((k_buckets<true, POL_PLAIN, kBucketUnroll>), dim3(uint32_t(grid)), dim3(kThreads), 0, st, sizes, rf, rb, cf, s.nranks, B, tptr, bptr);
  } else {
    if (ntm) hipLaunchKernelGGL((k_buckets<false, POL_NT, kBucketUnroll>), dim3(uint32_t(grid)), dim3(kThreads), 0, st, sizes, rf, rb, cf, s.nranks, B, tptr, bptr);
    else hipLaunchKernelGGL((k_buckets<false, POL_PLAIN, kBucketUnroll>), dim3(uint32_t(grid)), dim3(kThreads), 0, st, sizes, rf, rb, cf, s.nranks, B, tptr, bptr);
  }
  return hip_check(unpack ? "emu_unpack_buckets launch" : "emu_pack_buckets launch");
}

// Launches the reshard of plan P, whose tables (segments, tile map) start at device address w, for
// `groups` tensor groups.
static int launch_plan(const Plan* P, const uint8_t* w, const uint64_t* sp, const uint64_t* dp, uint32_t groups,
                       hipStream_t st, const char* what) {
  const LaunchRule rule = reshard_rule(*P, groups);
  const ReshardLaunch l{reinterpret_cast<const DevSeg*>(w + P->ws.off_segs),
                        reinterpret_cast<const uint32_t*>(w + P->ws.off_tilemap), P->ws.n_map, rule.cap, rule.blocks,
                        Tables{sp, dp, groups, uint32_t(P->side[0].tensors.size()), uint32_t(P->side[1].tensors.size())}, st};
  drop_pending_error();
  switch (P->tile_vecs) {
    case 1: launch_convert<1>(P->cvt, rule.policy, l); break;
    case 2: launch_convert<2>(P->cvt, rule.policy, l); break;
    case 4: launch_convert<4>(P->cvt, rule.policy, l); break;
    case 16: launch_convert<16>(P->cvt, rule.policy, l); break;
    default: launch_convert<8>(P->cvt, rule.policy, l); break;
  }
  return hip_check(what);
}

// Enqueue on st the plan's tables into device memory at `base` laid out as the workspace: the copies of
// the host-filled parts, then the kernels that derive the tile map and, with `sides`, each side's stream
// tables. Without `sides` only the workspace's first ws.reshard_bytes (all emu_reshard reads) are written.
static int enqueue_tables(const Plan* P, uint8_t* base, bool sides, hipStream_t st, const char* what) {
  const WsLayout& w = P->ws;
  const uint64_t head = w.off_tilemap;
  if (head) {
    const hipError_t e = hipMemcpyAsync(base, P->host_ws.data(), head, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return fail(EMU_ERR_HIP, "%s: segment upload: %s", what, hipGetErrorString(e));
  }
  if (sides && w.host_end > w.reshard_bytes) {
    const hipError_t e = hipMemcpyAsync(base + w.reshard_bytes, P->host_ws.data() + head, w.host_end - w.reshard_bytes,
                                        hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return fail(EMU_ERR_HIP, "%s: table upload: %s", what, hipGetErrorString(e));
  }
  drop_pending_error();
  if (w.n_map) {
    uint32_t longest = 0;
    for (uint32_t n : P->seg_tiles) longest = n > longest ? n : longest;
    const uint32_t gy = uint32_t(std::max<uint64_t>(1, std::min<uint64_t>(64, (uint64_t(longest) + 255) / 256)));
    hipLaunchKernelGGL(k_tile_map, dim3(uint32_t(P->dsegs.size()) + 1, gy), dim3(256), 0, st,
                       reinterpret_cast<const DevSeg*>(base + w.off_segs),
                       reinterpret_cast<const uint32_t*>(base + w.off_seg_tiles), uint32_t(P->dsegs.size()),
                       reinterpret_cast<uint32_t*>(base + w.off_tilemap), P->ntiles_copy, P->zero_tile0,
                       P->zero_tile0 + P->ntiles_zero, w.n_map);
  }
  for (int sd = 0; sides && sd < 2; ++sd) {
    const SideInfo& s = P->side[sd];
    const SideTables& t = w.side[sd];
    if (s.nranks <= 0) continue;
    const uint32_t* rf = reinterpret_cast<const uint32_t*>(base + t.off_rank_first);
    const uint64_t* rb = reinterpret_cast<const uint64_t*>(base + t.off_rank_bytes);
    uint64_t* so = reinterpret_cast<uint64_t*>(base + t.off_stream);
    uint64_t* ri = reinterpret_cast<uint64_t*>(base + t.off_rank_info);
    hipLaunchKernelGGL(k_stream_tables, dim3(uint32_t(s.nranks)), dim3(64), 0, st,
                       reinterpret_cast<const uint64_t*>(base + t.off_sizes), rf, rb, so, ri);
    if (t.n_tiles)  // an encodable side: at most 2^20 tensors
      hipLaunchKernelGGL(k_chunk_map, dim3(uint32_t(s.tensors.size()) + 1), dim3(256), 0, st, rf, rb,
                         uint32_t(s.nranks), uint32_t(s.tensors.size()), so, ri,
                         reinterpret_cast<uint32_t*>(base + t.off_tile_map), t.n_tiles);
  }
  return hip_check(what);
}

// ------------------------------------------------------------------------------------------------
// plan tables without a caller workspace (emu_reshard_noalloc)
// ------------------------------------------------------------------------------------------------
// For callers that cannot allocate device memory, the reshard tables go to a static device array. Each
// device the library runs on holds its own copy of the array, at its own address, until the process
// ends. Host code never uses the array's name as an address (in host code it names a host-side
// stand-in): once per device, with that device current, hipGetSymbolAddress gives the device address,
// which is kept per device and used for the upload and as the kernels' table pointer.
constexpr uint64_t kScratchBytes = 32ull << 20;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
struct ScratchSlot {
  std::mutex mu;
  void* ptr = nullptr;    // device address of `scratch` on this device
  uint64_t resident = 0;  // id of the plan whose tables the array holds (0: none)
};
static ScratchSlot g_scratch[kMaxDevices];

// The current device's array, holding P's tables: the first call on a device looks the array up, and
// the tables are copied in (on stream st) unless the array already holds them from an earlier call.
static int scratch_tables(const Plan* P, hipStream_t st, void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return fail(EMU_ERR_HIP, "cannot query the current device");
  if (dev < 0 || dev >= kMaxDevices) return fail(EMU_ERR_UNSUPPORTED, "device %d: at most %d devices", dev, kMaxDevices);
  ScratchSlot& sl = g_scratch[dev];
  std::lock_guard<std::mutex> lk(sl.mu);
  if (!sl.ptr) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail(EMU_ERR_HIP, "scratch address on device %d: %s", dev, hipGetErrorString(e));
    sl.ptr = p;
  }
  if (sl.resident != P->id) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
      return fail(EMU_ERR_ARG, "the static scratch does not hold this plan's tables: make one call outside stream "
                  "capture first");
    sl.resident = 0;
    if (int rc = enqueue_tables(P, static_cast<uint8_t*>(sl.ptr), false, st, "emu_reshard_noalloc tables")) return rc;
    sl.resident = P->id;
  }
  *out = sl.ptr;
  return EMU_OK;
}

}  // namespace emu

using namespace emu;

extern "C" {

int emu_plan_upload(emu_plan_t plan, void* d_workspace, uint64_t workspace_bytes, void* hip_stream) {
  clear_error();
  const Plan* P = reinterpret_cast<const Plan*>(plan);
  if (!plan_live(P)) return fail(EMU_ERR_HANDLE, "not a live plan");
  if (!d_workspace) return fail(EMU_ERR_NULL, "workspace is NULL");
  if (misaligned(d_workspace, kWsAlign)) return fail(EMU_ERR_WORKSPACE, "workspace not %llu-byte aligned", (unsigned long long)kWsAlign);
  if (workspace_bytes < P->ws.total)
    return fail(EMU_ERR_WORKSPACE, "workspace of %llu bytes, plan needs %llu", (unsigned long long)workspace_bytes,
                (unsigned long long)P->ws.total);
  ws_register(d_workspace, nullptr);  // until this upload is enqueued whole, the address holds no plan's tables
  if (int rc = enqueue_tables(P, static_cast<uint8_t*>(d_workspace), true, static_cast<hipStream_t>(hip_stream),
                              "emu_plan_upload"))
    return rc;
  ws_register(d_workspace, P);
  return EMU_OK;
}

int emu_reshard(emu_plan_t plan, const void* d_workspace, const uint64_t* d_src_ptrs, const uint64_t* d_dst_ptrs,
                void* hip_stream) {
  clear_error();
  const Plan* P = reinterpret_cast<const Plan*>(plan);
  if (!plan_live(P)) return fail(EMU_ERR_HANDLE, "not a live plan");
  if (!d_workspace || !d_src_ptrs || !d_dst_ptrs) return fail(EMU_ERR_NULL, "NULL workspace or pointer table");
  if (misaligned(d_workspace, kWsAlign)) return fail(EMU_ERR_WORKSPACE, "workspace not %llu-byte aligned", (unsigned long long)kWsAlign);
  if (misaligned(d_src_ptrs, 8) || misaligned(d_dst_ptrs, 8)) return fail(EMU_ERR_ALIGN, "pointer tables must be 8-byte aligned");
  if (P->ntiles == 0) return EMU_OK;
  if (!ws_current(d_workspace, P))
    return fail(EMU_ERR_WORKSPACE, "workspace %p holds no upload of this plan (fill it with emu_plan_upload)",
                d_workspace);
  return launch_plan(P, static_cast<const uint8_t*>(d_workspace), d_src_ptrs, d_dst_ptrs, 1,
                     static_cast<hipStream_t>(hip_stream), "emu_reshard launch");
}

int emu_reshard_groups(emu_plan_t plan, const void* d_workspace, int32_t n_groups, const uint64_t* d_src_ptrs,
                       const uint64_t* d_dst_ptrs, void* hip_stream) {
  clear_error();
  const Plan* P = reinterpret_cast<const Plan*>(plan);
  if (!plan_live(P)) return fail(EMU_ERR_HANDLE, "not a live plan");
  if (!d_workspace || !d_src_ptrs || !d_dst_ptrs) return fail(EMU_ERR_NULL, "NULL workspace or pointer table");
  if (n_groups < 1 || n_groups > 65535) return fail(EMU_ERR_RANGE, "n_groups %d not in [1, 65535]", n_groups);
  if (misaligned(d_workspace, kWsAlign)) return fail(EMU_ERR_WORKSPACE, "workspace not %llu-byte aligned", (unsigned long long)kWsAlign);
  if (misaligned(d_src_ptrs, 8) || misaligned(d_dst_ptrs, 8)) return fail(EMU_ERR_ALIGN, "pointer tables must be 8-byte aligned");
  if (P->ntiles == 0) return EMU_OK;
  if (!ws_current(d_workspace, P))
    return fail(EMU_ERR_WORKSPACE, "workspace %p holds no upload of this plan (fill it with emu_plan_upload)",
                d_workspace);
  return launch_plan(P, static_cast<const uint8_t*>(d_workspace), d_src_ptrs, d_dst_ptrs, uint32_t(n_groups),
                     static_cast<hipStream_t>(hip_stream), "emu_reshard_groups launch");
}

int emu_reshard_noalloc(emu_plan_t plan, const uint64_t* d_src_ptrs, const uint64_t* d_dst_ptrs, void* hip_stream) {
  clear_error();
  const Plan* P = reinterpret_cast<const Plan*>(plan);
  if (!plan_live(P)) return fail(EMU_ERR_HANDLE, "not a live plan");
  if (!d_src_ptrs || !d_dst_ptrs) return fail(EMU_ERR_NULL, "NULL pointer table");
  if (misaligned(d_src_ptrs, 8) || misaligned(d_dst_ptrs, 8)) return fail(EMU_ERR_ALIGN, "pointer tables must be 8-byte aligned");
  if (P->ntiles == 0) return EMU_OK;
  if (P->ws.reshard_bytes > kScratchBytes)
    return fail(EMU_ERR_WORKSPACE, "the plan's tables take %llu bytes, the static scratch holds %llu: use emu_reshard "
                "with a workspace", (unsigned long long)P->ws.reshard_bytes, (unsigned long long)kScratchBytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  void* w = nullptr;
  const int rc = scratch_tables(P, st, &w);
  if (rc) return rc;
  return launch_plan(P, static_cast<const uint8_t*>(w), d_src_ptrs, d_dst_ptrs, 1, st, "emu_reshard_noalloc launch");
}

int emu_pack_buckets(emu_plan_t plan, const void* d_workspace, int32_t side, uint64_t bucket_bytes,
                     const uint64_t* d_tensor_ptrs, const uint64_t* d_bucket_ptrs, void* hip_stream) {
  return bucket_call(plan, d_workspace, side, bucket_bytes, d_tensor_ptrs, d_bucket_ptrs, hip_stream, false);
}

int emu_unpack_buckets(emu_plan_t plan, const void* d_workspace, int32_t side, uint64_t bucket_bytes,
                       const uint64_t* d_bucket_ptrs, const uint64_t* d_tensor_ptrs, void* hip_stream) {
  return bucket_call(plan, d_workspace, side, bucket_bytes, d_tensor_ptrs, d_bucket_ptrs, hip_stream, true);
}

}  // extern "C"
