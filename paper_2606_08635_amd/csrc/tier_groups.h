// Tier-map bookkeeping shared by pack (which writes the map and the chunk
// index) and unpack (which checks them), one workgroup per map: a thread takes
// groups of 16 consecutive tokens, one map word each, eight loads in flight;
// the 16 groups of a 256-token chunk sit in 16 consecutive lanes, so chunk
// counts are a 16-lane reduction and the chunk index one block scan of them.
// Counting token by token with shared-memory atomics for the totals took
// pack_prep / unpack_check 7.2 / 7.2 us at 512 tokens, 8.5 / 8.2 at 4096 and
// 49 / 43 at 262144; this form takes 5.7 / 5.6, 5.7 / 5.5 and 18 / 11.
#pragma once

#include "device_util.h"
#include "skv_internal.h"

namespace skv {

constexpr int kGroupTokens = 16;
constexpr int kGroupsPerChunk = kChunkTokens / kGroupTokens;  // 16

// Tier counts of a run of tokens; the rest are FP16.
struct TierCounts {
  uint32_t n8, n4, nd;
};

// Row widths of `tokens` tokens in units of d/2 bytes: 4, 2, 1, 0 for FP16,
// INT8, INT4, DROP.
__device__ __forceinline__ uint32_t count_units(uint32_t tokens, TierCounts c) {
  return 4u * tokens - 2u * c.n8 - 3u * c.n4 - 4u * c.nd;
}

// Counts of at most 256 tokens and a flag count of at most 16, packed so that
// the 16 groups of a chunk add up without carries: INT8 in bits 0-8, INT4 in
// 9-17, DROP in 18-26, groups with a code outside 0..3 in 27-31.
__device__ __forceinline__ TierCounts unpack_counts(uint32_t p) {
  return TierCounts{p & 511u, (p >> 9) & 511u, (p >> 18) & 511u};
}
__device__ __forceinline__ bool counts_bad(uint32_t p) { return (p >> 27) != 0u; }

// Packed counts of the first `tokens` (0..16) codes of a 2-bit map word: a
// dozen bit operations and three population counts instead of a step per
// token.
__device__ __forceinline__ uint32_t map_word_counts(uint32_t w, int tokens) {
  const uint32_t valid = static_cast<uint32_t>((1ull << (2 * tokens)) - 1ull) & 0x55555555u;
  const uint32_t lo = w & valid, hi = (w >> 1) & valid;
  return static_cast<uint32_t>(__popc(lo & ~hi)) | static_cast<uint32_t>(__popc(hi & ~lo)) << 9 |
         static_cast<uint32_t>(__popc(lo & hi)) << 18;
}

// Four tier bytes as 8 map bits; codes outside 0..3 keep their low two bits.
__device__ __forceinline__ uint32_t map_byte(uint32_t w) {
  w &= 0x03030303u;
  return (w | w >> 6 | w >> 12 | w >> 18) & 0xFFu;
}

// The map word of a whole group of 16 tier bytes; bad: a code outside 0..3.
__device__ __forceinline__ uint32_t map_from_tiers(u32x4 t, bool& bad) {
  bad = ((t.x | t.y | t.z | t.w) & 0xFCFCFCFCu) != 0u;
  return map_byte(t.x) | map_byte(t.y) << 8 | map_byte(t.z) << 16 | map_byte(t.w) << 24;
}

// Tokens of group g of an n-token row (0 past its end).
__device__ __forceinline__ int group_tokens(int n, int g) { return min(kGroupTokens, max(0, n - g * kGroupTokens)); }

// The 16 tier bytes of group g, or the tokens there are, zero-filled.  The
// row may start at any byte; the last group of a row of at least 16 tokens is
// one load that ends with the row.
__device__ __forceinline__ u32x4 load_tiers(const uint8_t* __restrict__ tier, int n, int g) {
  typedef uint64_t u64x2_any __attribute__((ext_vector_type(2), aligned(1)));
  const int m = group_tokens(n, g);
  uint64_t lo = 0, hi = 0;
  if (m > 0 && n >= kGroupTokens) {
    const int over = kGroupTokens - m;  // bytes of the tokens before the group
    const u64x2_any w = *reinterpret_cast<const u64x2_any*>(tier + static_cast<size_t>(g) * kGroupTokens - over);
    lo = over == 0 ? w.x : over < 8 ? (w.x >> (8 * over)) | (w.y << (64 - 8 * over)) : w.y >> (8 * over - 64);
    hi = over < 8 ? w.y >> (8 * over) : 0ull;
  } else {
    for (int j = 0; j < m; ++j) {
      const uint64_t b = static_cast<uint64_t>(tier[j]) << (8 * (j & 7));
      if (j < 8) lo |= b;
      else hi |= b;
    }
  }
  return u32x4{static_cast<uint32_t>(lo), static_cast<uint32_t>(lo >> 32), static_cast<uint32_t>(hi),
               static_cast<uint32_t>(hi >> 32)};
}

// Sum over aligned 16-lane groups (the DPP rows); every lane gets its group's
// sum: quad swaps leave each lane its quad's sum, then the half-row mirror
// (lane i <-> 7 - i) pairs the quads of each half and the row mirror
// (i <-> 15 - i) the halves.  Every lane of the row must be active.
__device__ __forceinline__ uint32_t sum16(uint32_t v) {
  v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);  // row_half_mirror
  v += dpp_mov<0x140>(v);  // row_mirror
  return v;
}

constexpr int kMapThreads = 1024;  // of the kernels that write or check a tier map
constexpr int kMapBatch = 8;       // groups (or map words) per thread whose loads are in flight

// Counts of kMapBatch * kMapThreads groups of a tier array from group `base`
// on into s_chunk; map[k] receives the map word of group base + k *
// kMapThreads + thread.  Every thread of the block must call it.
__device__ __forceinline__ void tally_tiers(const uint8_t* __restrict__ tier, int n, int ngroups, int base,
                                            uint32_t* s_chunk, uint32_t (&map)[kMapBatch]) {
  u32x4 w[kMapBatch];
#pragma unroll
  for (int k = 0; k < kMapBatch; ++k) {
    w[k] = u32x4{0u, 0u, 0u, 0u};
    if (base + k * kMapThreads < ngroups)  // block-uniform
      w[k] = load_tiers(tier, n, base + k * kMapThreads + static_cast<int>(threadIdx.x));
  }
#pragma unroll
  for (int k = 0; k < kMapBatch; ++k) {
    map[k] = 0u;
    if (base + k * kMapThreads >= ngroups) continue;  // block-uniform
    const int g = base + k * kMapThreads + static_cast<int>(threadIdx.x);
    bool bad;
    map[k] = map_from_tiers(w[k], bad);
    const uint32_t c = sum16(map_word_counts(map[k], group_tokens(n, g)) | (bad ? 1u << 27 : 0u));
    if ((threadIdx.x % kGroupsPerChunk) == 0 && g < ngroups) s_chunk[g / kGroupsPerChunk] = c;
  }
}

// The same from the words of a 2-bit map (codes of tokens >= n are ignored).
__device__ __forceinline__ void tally_map(const uint8_t* __restrict__ map, int n, int ngroups, int base,
                                          uint32_t* s_chunk) {
  const uint32_t* words = reinterpret_cast<const uint32_t*>(map);
  uint32_t w[kMapBatch];
#pragma unroll
  for (int k = 0; k < kMapBatch; ++k) {
    const int g = base + k * kMapThreads + static_cast<int>(threadIdx.x);
    w[k] = g < ngroups ? words[g] : 0u;
  }
#pragma unroll
  for (int k = 0; k < kMapBatch; ++k) {
    if (base + k * kMapThreads >= ngroups) continue;  // block-uniform
    const int g = base + k * kMapThreads + static_cast<int>(threadIdx.x);
    const uint32_t c = sum16(map_word_counts(w[k], group_tokens(n, g)));
    if ((threadIdx.x % kGroupsPerChunk) == 0 && g < ngroups) s_chunk[g / kGroupsPerChunk] = c;
  }
}

// Exclusive prefix sums of one TierCounts per thread over a kMapThreads block,
// its totals, and whether any thread's `bad` is set.  Contains one
// __syncthreads(); s is not written again before the caller's next barrier.
struct CountScan {
  TierCounts before, total;
  bool bad;
};
struct CountScanLds {
  uint32_t w[4][kMapThreads / 64];
};
__device__ __forceinline__ CountScan block_scan_counts(TierCounts x, bool bad, CountScanLds& s) {
  static_assert(kMapThreads / 64 == 16, "one wave total per lane of a DPP row");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const uint32_t i8 = wave_inclusive_scan(x.n8), i4 = wave_inclusive_scan(x.n4), id = wave_inclusive_scan(x.nd);
  const uint64_t any = __ballot(bad);
  if (lane == 63) {
    s.w[0][wave] = i8;
    s.w[1][wave] = i4;
    s.w[2][wave] = id;
    s.w[3][wave] = any != 0 ? 1u : 0u;
  }
  __syncthreads();
  uint32_t before[4], total[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int inc = static_cast<int>(row_inclusive_scan(s.w[j][lane & 15]));
    total[j] = static_cast<uint32_t>(__builtin_amdgcn_readlane(inc, 15));
    before[j] = wave == 0 ? 0u : static_cast<uint32_t>(__builtin_amdgcn_readlane(inc, wave - 1));
  }
  return CountScan{{before[0] + i8 - x.n8, before[1] + i4 - x.n4, before[2] + id - x.nd},
                   {total[0], total[1], total[2]},
                   total[3] != 0u};
}

// Sum of the chunks [c0, c1) of s_chunk.
__device__ __forceinline__ TierCounts sum_chunks(const uint32_t* s_chunk, int c0, int c1, bool& bad) {
  TierCounts t{0u, 0u, 0u};
  for (int c = c0; c < c1; ++c) {
    const TierCounts x = unpack_counts(s_chunk[c]);
    bad |= counts_bad(s_chunk[c]);
    t.n8 += x.n8;
    t.n4 += x.n4;
    t.nd += x.nd;
  }
  return t;
}

// Chunk-index entry {units, quantized rows} before chunk c.
__device__ __forceinline__ u32x2 index_entry(int c, TierCounts before) {
  return u32x2{count_units(static_cast<uint32_t>(c) * kChunkTokens, before), before.n8 + before.n4};
}

// Zero-fills bytes [b0, b1) of p, 4 bytes per store (both multiples of 4).
__device__ __forceinline__ void zero_range(uint8_t* p, uint64_t b0, uint64_t b1, int tid, int nthreads) {
  for (uint64_t b = b0 + 4ull * tid; b < b1; b += 4ull * nthreads) *reinterpret_cast<uint32_t*>(p + b) = 0u;
}

// Word i (0..63) of the 256-byte payload header of request r, as pack writes it
// (non-finite row count and status zero).  Layout: 0 magic, 1 version, 2..5
// L, H, d, n, 6 sinks, 7 tiers, 8..10 budget / first-ratio / decay bits,
// 11 score mode, 12..15 tier counts, 16..35 u64 budget units, used units,
// tier-map, chunk-index and layer-0 offsets, segment bytes, segment stride,
// scale bytes, layer stride, total bytes; 36 non-finite rows, 37 status,
// 38 tokens per chunk.
__device__ __forceinline__ uint32_t header_word(const BatchArgs& a, const ReqDesc& r, int i) {
  auto lo = [](uint64_t x) { return static_cast<uint32_t>(x); };
  auto hi = [](uint64_t x) { return static_cast<uint32_t>(x >> 32); };
  switch (i) {
    case 0: return kMagic;
    case 1: return kVersion;
    case 2: return static_cast<uint32_t>(a.L);
    case 3: return static_cast<uint32_t>(a.H);
    case 4: return static_cast<uint32_t>(a.d);
    case 5: return static_cast<uint32_t>(r.n);
    case 6: return static_cast<uint32_t>(r.n_sink);
    case 7: return static_cast<uint32_t>(a.num_tiers);
    case 8: return a.budget_bits;
    case 9: return a.rho_bits;
    case 10: return a.decay_bits;
    case 11: return static_cast<uint32_t>(a.score_mode);
    case 12: return static_cast<uint32_t>(r.n16);
    case 13: return static_cast<uint32_t>(r.n8);
    case 14: return static_cast<uint32_t>(r.n4);
    case 15: return static_cast<uint32_t>(r.nd);
    case 16: return lo(static_cast<uint64_t>(r.budget_units));
    case 17: return hi(static_cast<uint64_t>(r.budget_units));
    case 18: return lo(static_cast<uint64_t>(r.used_units));
    case 19: return hi(static_cast<uint64_t>(r.used_units));
    case 20: return 256u;  // tier map right after the header
    case 21: return 0u;
    case 22: return lo(r.chunkidx_off);
    case 23: return hi(r.chunkidx_off);
    case 24: return lo(r.layers_off);
    case 25: return hi(r.layers_off);
    case 26: return lo(r.seg_bytes);
    case 27: return hi(r.seg_bytes);
    case 28: return lo(r.seg_stride);
    case 29: return hi(r.seg_stride);
    case 30: return lo(r.scales_bytes);
    case 31: return hi(r.scales_bytes);
    case 32: return lo(r.layer_stride);
    case 33: return hi(r.layer_stride);
    case 34: return lo(r.total);
    case 35: return hi(r.total);
    case 38: return static_cast<uint32_t>(kChunkTokens);
    case 39: return static_cast<uint32_t>(a.q8);
    case 40: return static_cast<uint32_t>(a.q4);
    case 42: return lo(r.channel_bytes);
    case 43: return hi(r.channel_bytes);
    default: return 0u;
  }
}
constexpr int kHdrNonfinite = 36;
constexpr int kHdrStatus = 37;

// The request that owns flat (segment, chunk) pair `bid` of a batched row
// launch: all starts are one scalar load (looking them up in the descriptors,
// one load each, cost a workgroup of a sixteen-request launch more than its
// scan).
__device__ __forceinline__ int request_of_block(const BatchArgs& a, uint32_t bid) {
  int r = 0;
  if (a.count > 1) {
#pragma unroll
    for (int i = 1; i < kMaxBatch; ++i) r = a.begin[i] <= bid ? i : r;
  }
  return r;
}

// Place of flat (segment, chunk) pair `local` of request r: segments are
// ((l - layer_begin) * 2 + kv) * H + h, chunk fastest.
struct RowPlace {
  int chunk, h, kv, l;
};
__device__ __forceinline__ RowPlace row_place(const BatchArgs& a, const ReqDesc& r, uint32_t local) {
  const uint32_t seg = r.by_chunks.div(local), lkv = a.by_heads.div(seg);
  return RowPlace{static_cast<int>(local - seg * static_cast<uint32_t>(r.nchunks)),
                  static_cast<int>(seg - lkv * static_cast<uint32_t>(a.H)), static_cast<int>(lkv & 1u),
                  a.layer_begin + static_cast<int>(lkv >> 1)};
}

// The same for launches over the chunks of only the K or only the V segments:
// pair `local` counts (layer, head, chunk), chunk fastest.
__device__ __forceinline__ RowPlace side_place(const BatchArgs& a, const ReqDesc& r, uint32_t local, int kv) {
  const uint32_t seg = r.by_chunks.div(local), l = a.by_heads.div(seg);
  return RowPlace{static_cast<int>(local - seg * static_cast<uint32_t>(r.nchunks)),
                  static_cast<int>(seg - l * static_cast<uint32_t>(a.H)), kv, a.layer_begin + static_cast<int>(l)};
}

}  // namespace skv
