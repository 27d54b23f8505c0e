// The per-chunk bodies of the row kernels, shared by the per-token codec
// (pack.hip, unpack.hip) and the grouped codec (groups.hip): workgroups of
// 256 threads own a 256-token chunk of one (layer, K/V, head) segment, one or
// several of them (SPLIT) an equal run of its tokens each.
//   chunk_layout_*  give every token of the chunk its tier, the byte offset
//                   of its row inside the segment and the index of its scale
//                   (chunk-index base + a block scan of the row widths);
//   pack_load / pack_store
//                   read the rows (d/8 lanes per row, 16 bytes each, all of a
//                   thread's rows in flight before the layout scan), quantize
//                   and store them;
//   unpack_chunk    loads the rows at their tier widths, dequantizes and
//                   writes them into their paged slots.
#pragma once

#include "device_util.h"
#include "row_codec.h"
#include "skv_internal.h"

namespace skv {

// Workgroups that share a chunk in the default-quantizer row kernels (measured
// on MI355X; pack, then unpack, us, one workgroup per chunk with 8 or 16 rows
// in flight per thread against the split below).
// Pack takes 4 rows per thread, all in flight at once, and no loop: 36 VGPRs
// instead of 96, so eight waves per SIMD instead of five, and shorter
// workgroups, so a shorter last wave (32 x 8 x 128 x 32768 1047 -> 993, x 8189
// 279 -> 256, 28 x 4 x 128 x 4096 74 -> 65, 42 x 8 x 256 x 8192 718 -> 646,
// 32 x 8 x 64 x 32768 520 -> 499).  2 rows: 15-20 % slower.
// Unpack takes 4 rows at d = 128 (1181 -> 1103, 304 -> 291, 80 -> 72); at
// d = 256 16 rows, two batches, stream better in long launches (42 x 8 x 256 x
// 8192 749 against 771-785) and 8 rows, one batch, in launches of at most 6144
// chunks (x 2048 204 -> 186, 10 x 8 x 256 x 4096 106 -> 101); at d = 64 and 32
// a chunk is 8 and 4 rows per thread and is not split, except in launches of at
// most 512 chunks, two for each CU, where 2 rows per thread with their scales
// save a round trip (check and rows at 8, 64, 512 and 1024 chunks, d = 64: 11.0 ->
// 8.5, 11.3 -> 9.0, 13.9 -> 13.4, but 16.5 -> 19.6; d = 32 at 8, 512 and 2048:
// 9.3 -> 8.5, 11.7 -> 11.1, but 19.7 -> 22.3).
// Both store non-temporally: default-policy stores leave up to the caches'
// size of dirty lines behind when the kernel ends, and the kernels after it
// pay their write-back (pack + unpack back to back: 2.7 % slower at d = 128,
// 1.7-2.9 % at d = 256).
template <int D>
constexpr int pack_split() { return D / 32; }
// The quantizer variants' pack is bound by vector instructions, so the layout
// scan that every workgroup repeats counts: 8 rows per thread in long launches
// (32 x 8 x 128 x 32768, asymmetric fp32 groups of 64: 1270 us with a workgroup
// per chunk, 1321 with 4 rows per thread, 1221 with 8; binary16 row scales 1187,
// 1158, 1062), 4 in short ones.
template <int D>
constexpr int pack_split_variant() { return D >= 128 ? D / 64 : 1; }
template <int D>
constexpr int unpack_split_long() { return D == 128 ? 4 : 1; }
template <int D>
constexpr int unpack_split_short() { return D >= 128 ? 4 : 1; }
template <int D>
constexpr int unpack_split_tiny() { return D == 32 ? 2 : 4; }
// Pack of requests of 129 to 192 tokens at d = 64, of up to 224 in launches that
// are not resident at once: one workgroup of 8 rows per thread, as a second one of 4
// is short of rows but takes a slot (prep and rows, us, a workgroup per chunk before,
// two, this: 80 x 8 pairs, 129 tokens 16.2, 17.2, 13.8, 160 tokens 17.0, 17.9, 14.8, 200
// tokens 19.4, 19.4, 16.4; 28 x 4 pairs, two and this, 193 tokens 11.1, 12.1; six requests
// of 80 x 8 pairs, 240 tokens 62, 65).
template <int D>
constexpr int pack_split_short() { return D == 64 ? 1 : pack_split<D>(); }
template <int D>
bool short_pack(int longest, uint64_t chunks) {
  return D == 64 && longest > kChunkTokens / 2 && longest <= (chunks > 1024 ? 224 : 192);
}
// Unpack of requests of 65 to 128 tokens at d = 128: one workgroup of 8 rows per
// thread.  Of two with 4 the second is short of rows but takes a slot all the same
// (check and rows, us, a workgroup per chunk, two, this: 80 x 8 pairs, 80 tokens
// 16.9, 17.6, 14.1, 128 tokens 20.8, 21.4, 18.3; 12 requests of 40 x 8 pairs, 65 tokens
// 53.7, 55.9, 45.6, 128 tokens 87.2, 81.2, 80.3; no difference up to 28 x 4 pairs).
template <int D>
constexpr int unpack_split_half() { return D == 128 ? 2 : unpack_split_short<D>(); }
template <int D>
bool half_chunks(int longest) { return D == 128 && longest <= kChunkTokens / 2 && longest > kChunkTokens / 4; }
// The quantizer variants (4 rows in flight) unpack long launches best with two
// workgroups per chunk (one, two, four: 32 x 8 x 128 x 8192 318 / 313 / 318,
// 42 x 8 x 256 x 4096 per-channel keys 485 / 458 / 477) and short ones with
// four (4 x 4 x 128 x 1000 24.6 / 17.1 / 13.7, 28 x 4 x 128 x 4096 88 / 81 / 78).
template <int D>
constexpr int unpack_split_variant() { return D >= 128 ? 2 : 1; }
constexpr uint64_t kShortLaunch = 6144;  // chunks
// Per-channel keys at d = 256: each part of a chunk checks and loads all of its
// channel entries, and the parts of a chunk of a long segment do so on different
// XCDs.  Between these launch sizes a segment of more than 64 chunks therefore takes
// one workgroup per chunk (four and one, asymmetric binary16 | symmetric binary32, us:
// 2 x 8 x 31803 222, 185 | 200, 177; 1 x 8 x 60000 225, 198 | 208, 175; 4 x 8 x 17000
// 220, 205 | 191, 204).  Below, too few workgroups are left (1 x 4 x 32768 63, 73 |
// 54, 68); above, two are as fast (8 x 8 x 17000 384, 384 | 363, 371); shorter
// segments are faster in parts (28 x 4 x 4096 167, two 176; one 207).
constexpr uint64_t kWholeLaunch = 3584;
template <int D>
bool whole_chunks(uint64_t chunks, uint64_t segments) {
  return D == 256 && chunks > kWholeLaunch && chunks <= kShortLaunch && chunks > 64 * segments;
}
constexpr uint64_t kTinyLaunch = 512;
constexpr int kUnpackRowsInFlight = 16;
// The quantizer-variant kernels hold more per row (group metadata): 4 rows.
#ifndef SKV_VAR_ROWS_IN_FLIGHT
#define SKV_VAR_ROWS_IN_FLIGHT 4
#endif

// The flat index of this workgroup when runs of kXcdRun consecutive indexes
// share an XCD (workgroups are dealt to the eight XCDs in turn; the last,
// incomplete round of 8 runs keeps its order).  Pack: neighbouring workgroups'
// rows and scales meet in one L2 (24 requests of 100-2300 tokens, 32 x 8 x 128:
// encode + decode 2024 -> 1959 us, 28 x 4 x 128 x 4096 180 -> 172, 32 x 8 x 128
// x 32768 2899 -> 2855; runs of 4 and 8 lose 2-3 % there, runs of 512 gain
// half), but not in launches that are resident at once (512 chunks of 28 x 4 x
// 128 x 4096: 1 % slower).  Unpack: only where a segment is at most kXcdRun workgroups long, so
// that a run writes neighbouring heads of the same slots (the batch 2024 ->
// 1972, 4096 tokens 180 -> 174; from 8189 tokens on 1 % slower).
constexpr uint32_t kXcdRun = 64;
constexpr uint32_t kXcdLeast = 4096;  // workgroups: more than the GPU holds at once
// `first`: the flat index of the launch's first workgroup (launch_pieces).
__device__ __forceinline__ uint32_t xcd_block(uint32_t first) {
  const uint32_t b = blockIdx.x, round = b & ~(8u * kXcdRun - 1u);
  return first + (gridDim.x >= kXcdLeast && round + 8u * kXcdRun <= gridDim.x ? round + (b & 7u) * kXcdRun + ((b - round) >> 3) : b);
}

// A chunk's parts.  A part of SPLIT that starts past the last token has nothing to
// do, and the workgroup that owns it leaves early.  Launches whose requests have
// one chunk each make only as many parts as hold tokens, a power of two of them
// (log2).  Where such parts remain (last chunks, batches of unlike lengths),
// workgroups are dealt to XCDs and within them in turn, so the parts that do have
// tokens would all meet on a few: `turned`, a chunk's parts begin at a place that a
// hash of its index scatters.  Without either, a short request's rows fell on 2 of
// 8 XCDs (80 x 8 x 128: one workgroup per chunk, four in fixed order, now, us:
// unpack of 20 tokens 13.8, 16.9, 10.6, of 64 tokens 16.0, 23.5, 13.3, of 12
// requests of 20 tokens 69, 131, 44; pack 15.4, 17.0, 10.8, then 18.2, 23.6, 13.5
// and 96, 127, 43; 24 requests of 17-316 tokens, 32 x 8 x 128, pack 217, 193, 154
// and unpack 200, 223, 170).  Whole chunks and segments of more than 8, where a
// last chunk weighs little, keep the fixed order.  Fixed against turned, us: 28 x 4
// x 128, unpack of 520 tokens 18.8, 17.2, of 1150 28.4, 26.5, pack of 2300 40.8, 41.0
// and of 4000 63.1, 63.8; 28 x 4 x 128 x 4096, pack, link and unpack four layers at a
// time, 244.6, 248.5; unpack of 32 x 8 x 128 x 32768 1151, 1165.
struct ChunkParts {
  uint32_t log2;
  bool turned;
};
__device__ __forceinline__ int chunk_part(uint32_t block, ChunkParts p) {
  const uint32_t turn = p.turned ? (block >> p.log2) * 0x9E3779B1u >> 24 : 0u;
  return static_cast<int>((block + turn) & ((1u << p.log2) - 1u));
}
constexpr int kTurnedChunks = 8;
inline bool turned_parts(int n) { return n % kChunkTokens != 0 && n <= kTurnedChunks * kChunkTokens; }
inline bool turned_parts(const BatchArgs& a) {
  for (int i = 0; i < a.count; ++i)
    if (turned_parts(a.r[i].n)) return true;
  return false;
}
// The parts that a launch makes of a chunk; longest: its longest request.
template <int SPLIT>
ChunkParts launch_parts(int longest, bool turned) {
  ChunkParts p{0, turned};
  while ((1 << p.log2) < SPLIT && longest > (kChunkTokens / SPLIT << p.log2)) ++p.log2;
  return p;
}

constexpr int kRowThreads = 256;  // == kChunkTokens: one token per thread in the scan
static_assert(kRowThreads == kChunkTokens, "one scan slot per token of a chunk");
constexpr int kAbsent = 4;  // unpack: a slot past the end of the request

struct ChunkLds {
  uint8_t tier[kChunkTokens];
  uint32_t off[kChunkTokens];  // byte offset of the row inside its segment
  uint32_t q[kChunkTokens];    // index of the row's scale
  uint32_t pos[kChunkTokens];  // unpack: physical block * block_size + slot
  float scale[kChunkTokens];   // unpack: the row's scale (quantized rows)
  uint32_t scan[4];
};

// Unpack, whole chunks: stages the scale of the chunk's row of this thread's
// scan slot (tier code tr) in shared memory, read with one load per quantized
// row rather than one per lane of each row.  The scale index is this thread's
// own s.q entry; the caller's barrier after chunk_layout publishes it.
__device__ __forceinline__ void stage_scale(ChunkLds& s, int tr, const float* __restrict__ scales) {
  s.scale[threadIdx.x] = (tr == kINT8 || tr == kINT4) ? scales[s.q[threadIdx.x]] : 0.0f;
}

// Fills s.tier/off/q of the chunk starting at t0 from the token's tier code
// tr (kDROP for pack slots past n, kAbsent for unpack slots past n) and the
// chunk's index entry {units, quantized rows}.  Contains __syncthreads().
template <int D>
__device__ __forceinline__ void chunk_layout(ChunkLds& s, int tr, const uint32_t* cidx_entry) {
  const uint32_t packed = tier_units(tr) | (tier_quant(tr) << 16);
  const uint32_t ex = block_exclusive_scan_256(packed, s.scan);
  s.tier[threadIdx.x] = static_cast<uint8_t>(tr);
  s.off[threadIdx.x] = (cidx_entry[0] + (ex & 0xFFFFu)) * static_cast<uint32_t>(D / 2);
  s.q[threadIdx.x] = cidx_entry[1] + (ex >> 16);
}

// Rows of one thread: lanes per row (16 bytes each), rows per block-wide
// iteration, iterations of a workgroup's part of the chunk (part `sub` of
// SPLIT starts at token sub * ITERS * RPI), rows in flight.
template <int D, int ROWS_IN_FLIGHT, int SPLIT>
struct RowBatch {
  static constexpr int LPR = D / 8;
  static constexpr int RPI = kRowThreads / LPR;
  static constexpr int ITERS = kChunkTokens / RPI / SPLIT;
  static constexpr int U = ITERS < ROWS_IN_FLIGHT ? ITERS : ROWS_IN_FLIGHT;
  static_assert(ITERS > 0 && ITERS % U == 0, "rows in flight must divide a thread's rows of the chunk");
};
template <int D, int SPLIT>
struct PackRows : RowBatch<D, 8, SPLIT> {
  static_assert(PackRows::U == PackRows::ITERS, "one batch");
  u32x4 x[PackRows::U];
};

// Issues the loads of a thread's rows of the chunk at t0, taking their tiers
// from the caller's tier map (tier[t], t < n) rather than from the chunk
// layout: the loads are then in flight while the layout is scanned.  Reads
// only rows t < n of tiers other than DROP.
template <int D, int SPLIT>
__device__ __forceinline__ void pack_load(PackRows<D, SPLIT>& b, const uint16_t* __restrict__ src,
                                          const uint8_t* __restrict__ tier, int t0, int n, int sub) {
  using B = PackRows<D, SPLIT>;
  const int lane = threadIdx.x % B::LPR;
  const int t1 = t0 + sub * B::ITERS * B::RPI + threadIdx.x / B::LPR;
  uint8_t tr[B::U];  // loaded together: one round trip
#pragma unroll
  for (int u = 0; u < B::U; ++u) tr[u] = tier[min(t1 + u * B::RPI, n - 1)];
#pragma unroll
  for (int u = 0; u < B::U; ++u) {
    const int t = t1 + u * B::RPI;
    b.x[u] = u32x4{0u, 0u, 0u, 0u};
    if (t < n && tr[u] != kDROP) b.x[u] = ld_nt16(src + static_cast<size_t>(t) * D + lane * 8);
  }
}

// Quantizes and stores the loaded rows.  dst: the segment's rows; scales: the
// segment's scales.
template <int D, int SPLIT>
__device__ __forceinline__ void pack_store(const ChunkLds& s, const PackRows<D, SPLIT>& b, uint8_t* __restrict__ dst,
                                           float* __restrict__ scales, uint32_t* nonfinite, int sub) {
  using B = PackRows<D, SPLIT>;
  const int lane = threadIdx.x % B::LPR;
  const int r1 = sub * B::ITERS * B::RPI + threadIdx.x / B::LPR;
#pragma unroll
  for (int u = 0; u < B::U; ++u) {
    const int row = r1 + u * B::RPI;
    const int tr = s.tier[row];
    const uint32_t amax = group_max<B::LPR>(absmax_bits8(b.x[u]));  // all lanes take part
    if (tr == kFP16) {
      st_nt16(dst + s.off[row] + lane * 16, b.x[u]);
    } else if (tr == kINT8 || tr == kINT4) {
      const LaneCodes q = quantize_lane(b.x[u], amax, tr == kINT8 ? 127 : 7);
      if (q.nonfinite && lane == 0) atomicAdd(nonfinite, 1u);
      uint8_t* out_row = dst + s.off[row];
      if (tr == kINT8) st_nt8(out_row + lane * 8, pack_int8(q));
      else st_nt4(out_row + lane * 4, pack_int4(q));
      if (lane == 0) scales[s.q[row]] = q.scale;
    }
  }
}

// Loads one row slice of a lane: 16 B of FP16, 8 B of INT8 codes or 4 B of
// INT4 codes.
__device__ __forceinline__ void load_row(int tr, const uint8_t* row, int lane, u32x4& raw) {
  raw = u32x4{0u, 0u, 0u, 0u};
  if (tr == kFP16) {
    raw = ld_nt16(row + lane * 16);
  } else if (tr == kINT8) {
    const u32x2 c = ld_nt8(row + lane * 8);
    raw.x = c.x;
    raw.y = c.y;
  } else if (tr == kINT4) {
    raw.x = ld_nt4(row + lane * 4);
  }
}

// The lane's 8 output elements of a row: FP16 verbatim, DROP zeros, INT8/INT4
// dequantized, a NaN scale giving 0x7E00 (and any NaN product, 0x7E00).
__device__ __forceinline__ u32x4 decode_row(int tr, u32x4 raw, float sc) {
  if (tr == kINT8 || tr == kINT4) {
    if (__builtin_isnan(sc)) return u32x4{kNaNHalf2, kNaNHalf2, kNaNHalf2, kNaNHalf2};
    const u32x4 o = tr == kINT8 ? dequant_int8(u32x2{raw.x, raw.y}, sc) : dequant_int4(raw.x, sc);
    // only an infinite scale makes a NaN product (code 0): written as 0x7E00
    return __builtin_isinf(sc) ? canon_nan_lane(o) : o;
  }
  return raw;
}

// Dequantizes a workgroup's rows of one chunk into their paged slots.  src: the
// segment's rows; scales: the segment's scales, staged in s.scale (stage_scale)
// where the workgroup owns the chunk and loaded with the rows (a round trip
// less) where it shares it; cache: the (layer, head) column of the paged cache
// (slot stride H * D elements).
template <int D, int SPLIT>
__device__ __forceinline__ void unpack_chunk(const ChunkLds& s, const uint8_t* __restrict__ src,
                                             const float* __restrict__ scales, uint16_t* __restrict__ cache, int H,
                                             int sub) {
  using B = RowBatch<D, D == 256 ? kUnpackRowsInFlight : 8, SPLIT>;
  constexpr int RPI = B::RPI, ITERS = B::ITERS, U = B::U;
  const int lane = threadIdx.x % B::LPR;
  const int r1 = sub * ITERS * RPI + threadIdx.x / B::LPR;
#pragma unroll 1
  for (int it = 0; it < ITERS; it += U) {
    u32x4 raw[U];
    float sc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r1 + (it + u) * RPI;
      const int tr = s.tier[r];
      load_row(tr, src + s.off[r], lane, raw[u]);
      if constexpr (SPLIT == 1) {
        sc[u] = s.scale[r];
      } else {
        sc[u] = 0.0f;
        if (tr == kINT8 || tr == kINT4) sc[u] = scales[s.q[r]];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r1 + (it + u) * RPI;
      const int tr = s.tier[r];
      if (tr == kAbsent) continue;
      st_nt16(cache + static_cast<size_t>(s.pos[r]) * H * D + lane * 8, decode_row(tr, raw[u], sc[u]));
    }
  }
}

}  // namespace skv
