// Per-layer and per-head tier maps (the extension named in Sec. 2.6,
// Sec. 6.10, Sec. 7.5 and Sec. 9 (iii)): the (layer, head) pairs are split
// into G groups, one per layer or one per (layer, head), and each group has
// its own budget, plan and tier map.  The grouped payload carries a group
// table, G tier maps and G chunk indexes, and a segment table with the
// offsets of every segment's scales and rows (segment sizes differ between
// groups).  Row work is the per-token codec's (row_stream.h); only the
// lookups of a segment's group, map, chunk index and offsets differ.
//   gpack_init    zeroes the header's non-finite counter and status words
//                 and the caller's status word;
//   gpack_prep    one workgroup per group checks the group's tier map against
//                 its plan and writes its 2-bit map and chunk index; one more
//                 workgroup writes the header, group table and segment table;
//   gpack_rows    one to d/32 workgroups per (segment, 256-token chunk), as
//                 pack_rows;
//   gunpack_init, gunpack_check (one workgroup per group + one for header
//                 and tables), gunpack_rows (one to four workgroups per
//                 (segment, chunk), as unpack_rows): the decode side.
#include "device_util.h"
#include "row_codec.h"
#include "row_stream.h"
#include "skv_internal.h"
#include "tier_groups.h"

namespace skv {
namespace {

constexpr int kMaxChunks = kMaxTokens / kChunkTokens;
constexpr uint32_t kGroupMagic = 0x47564B53u;  // "SKVG"
constexpr int kGHdrNonfinite = 32;
constexpr int kGHdrStatus = 33;

struct GroupArgs {
  const uint16_t* k;
  const uint16_t* v;
  const uint8_t* tier;          // pack: uint8 [G][n]
  uint8_t* payload;
  uint32_t* status;             // pack: optional; unpack: required
  const uint32_t* group_table;  // workspace: G x 8 words
  const uint64_t* segtab;       // workspace: 2LH x {scales offset, rows offset}
  const int32_t* block_table;
  int32_t num_blocks, block_size;
  int32_t L, H, d, n, gran, G, nchunks, num_tiers, score_mode, num_sink;
  uint32_t budget_bits, rho_bits, decay_bits;
  uint64_t group_off, tiermaps_off, tiermap_stride, chunkidx_off, chunkidx_stride, segtab_off, layers_off, total;
  Divider by_chunks, by_heads, by_block;  // by nchunks, H, block_size (unpack)
};

__device__ __forceinline__ int group_of(const GroupArgs& a, int l, int h) {
  return a.gran == SKV_GROUP_TOKEN ? 0 : a.gran == SKV_GROUP_LAYER ? l : l * a.H + h;
}

__device__ __forceinline__ uint32_t lo32(uint64_t x) { return static_cast<uint32_t>(x); }
__device__ __forceinline__ uint32_t hi32(uint64_t x) { return static_cast<uint32_t>(x >> 32); }

__device__ __forceinline__ uint32_t gheader_word(const GroupArgs& a, int i) {
  switch (i) {
    case 0: return kGroupMagic;
    case 1: return kVersion;
    case 2: return static_cast<uint32_t>(a.L);
    case 3: return static_cast<uint32_t>(a.H);
    case 4: return static_cast<uint32_t>(a.d);
    case 5: return static_cast<uint32_t>(a.n);
    case 6: return static_cast<uint32_t>(a.gran);
    case 7: return static_cast<uint32_t>(a.G);
    case 8: return static_cast<uint32_t>(a.num_tiers);
    case 9: return static_cast<uint32_t>(a.score_mode);
    case 10: return a.budget_bits;
    case 11: return a.rho_bits;
    case 12: return a.decay_bits;
    case 13: return static_cast<uint32_t>(a.num_sink);
    case 14: return static_cast<uint32_t>(kChunkTokens);
    case 16: return lo32(a.group_off);
    case 17: return hi32(a.group_off);
    case 18: return lo32(a.tiermaps_off);
    case 19: return hi32(a.tiermaps_off);
    case 20: return lo32(a.tiermap_stride);
    case 21: return hi32(a.tiermap_stride);
    case 22: return lo32(a.chunkidx_off);
    case 23: return hi32(a.chunkidx_off);
    case 24: return lo32(a.chunkidx_stride);
    case 25: return hi32(a.chunkidx_stride);
    case 26: return lo32(a.segtab_off);
    case 27: return hi32(a.segtab_off);
    case 28: return lo32(a.layers_off);
    case 29: return hi32(a.layers_off);
    case 30: return lo32(a.total);
    case 31: return hi32(a.total);
    default: return 0u;  // 15, the counters (32, 33) and the reserved words
  }
}

// Bytes of a group's segment rows (before padding).
__device__ __forceinline__ uint64_t group_seg_bytes(const uint32_t* e, int D) {
  return static_cast<uint64_t>(e[0] + e[1]) * (2 * D) + static_cast<uint64_t>(e[2]) * D +
         static_cast<uint64_t>(e[3]) * (D / 2);
}

__global__ void gpack_init(const GroupArgs a) {
  uint32_t* hdr = reinterpret_cast<uint32_t*>(a.payload);
  if (threadIdx.x == 0) {
    hdr[kGHdrNonfinite] = 0u;
    hdr[kGHdrStatus] = 0u;
    if (a.status) *a.status = 0u;
  }
}

// grid: G + 1 workgroups
__global__ __launch_bounds__(kMapThreads) void gpack_prep(const GroupArgs a) {
  __shared__ uint32_t s_chunk[kMaxChunks];
  __shared__ CountScanLds s_scan;
  uint8_t* __restrict__ payload = a.payload;
  const int tid = threadIdx.x;
  if (blockIdx.x == static_cast<unsigned>(a.G)) {
    // header (but the two counters), group table, segment table and their padding
    uint32_t* hdr = reinterpret_cast<uint32_t*>(payload);
    if (tid < 64 && tid != kGHdrNonfinite && tid != kGHdrStatus) hdr[tid] = gheader_word(a, tid);
    uint32_t* gt = reinterpret_cast<uint32_t*>(payload + a.group_off);
    for (int i = tid; i < 8 * a.G; i += kMapThreads) gt[i] = a.group_table[i];
    zero_range(payload, a.group_off + 32ull * a.G, a.tiermaps_off, tid, kMapThreads);
    uint64_t* st = reinterpret_cast<uint64_t*>(payload + a.segtab_off);
    const int nseg = 2 * a.L * a.H;
    for (int i = tid; i < 2 * nseg; i += kMapThreads) st[i] = a.segtab[i];
    zero_range(payload, a.segtab_off + 16ull * nseg, a.layers_off, tid, kMapThreads);
    return;
  }
  const int g = blockIdx.x;
  const uint32_t* e = a.group_table + 8 * g;
  const uint8_t* __restrict__ tier = a.tier + static_cast<size_t>(g) * a.n;
  const int n = a.n, nchunks = a.nchunks;
  const int ngroups = (n + kGroupTokens - 1) / kGroupTokens;
  constexpr int kBatch = kMapBatch * kMapThreads;
  uint32_t map0[kMapBatch];
  tally_tiers(tier, n, ngroups, 0, s_chunk, map0);
  for (int base = kBatch; base < ngroups; base += kBatch) {
    uint32_t rest[kMapBatch];
    tally_tiers(tier, n, ngroups, base, s_chunk, rest);
  }
  __syncthreads();
  // each thread owns a run of consecutive chunks
  const int per = (nchunks + kMapThreads - 1) / kMapThreads;
  const int c0 = min(nchunks, tid * per), c1 = min(nchunks, c0 + per);
  bool bad = false;
  const TierCounts mine = sum_chunks(s_chunk, c0, c1, bad);
  const CountScan sc = block_scan_counts(mine, bad, s_scan);
  const bool ok = !sc.bad && sc.total.n8 == e[2] && sc.total.n4 == e[3] && sc.total.nd == e[4];  // FP16 follows
  if (!ok) {  // block-uniform
    if (tid == 0) {
      atomicOr(reinterpret_cast<uint32_t*>(payload) + kGHdrStatus, static_cast<uint32_t>(SKV_ERR_INVALID_ARG));
      if (a.status) atomicOr(a.status, static_cast<uint32_t>(SKV_ERR_INVALID_ARG));
    }
    return;
  }
  // chunk index of the group (running sums at every chunk start) and padding
  const uint64_t ci_off = a.chunkidx_off + static_cast<uint64_t>(g) * a.chunkidx_stride;
  TierCounts at = sc.before;
  for (int c = c0; c < c1; ++c) {
    reinterpret_cast<u32x2*>(payload + ci_off)[c] = index_entry(c, at);
    const TierCounts x = unpack_counts(s_chunk[c]);
    at.n8 += x.n8;
    at.n4 += x.n4;
    at.nd += x.nd;
  }
  zero_range(payload, ci_off + 8ull * nchunks, ci_off + a.chunkidx_stride, tid, kMapThreads);
  // the group's 2-bit map (4 bytes per 16 tokens) and padding
  const uint64_t map_off = a.tiermaps_off + static_cast<uint64_t>(g) * a.tiermap_stride;
  uint32_t* map = reinterpret_cast<uint32_t*>(payload + map_off);
#pragma unroll
  for (int k = 0; k < kMapBatch; ++k) {
    const int q = k * kMapThreads + tid;
    if (q < ngroups) map[q] = map0[k];
  }
  for (int q = kBatch + tid; q < ngroups; q += kMapThreads) {
    bool b;
    map[q] = map_from_tiers(load_tiers(tier, n, q), b);
  }
  zero_range(payload, map_off + 4ull * ngroups, map_off + a.tiermap_stride, tid, kMapThreads);
}

// grid: 2^parts.log2 workgroups (pack_split<D>(), fewer where n is less than a
// chunk) for each of 2 * L * H * nchunks chunks, chunk fastest
template <int D>
__global__ __launch_bounds__(kRowThreads) void gpack_rows(const GroupArgs a, uint32_t first, ChunkParts parts) {
  __shared__ ChunkLds s;
  uint8_t* __restrict__ payload = a.payload;
  uint32_t* hdr = reinterpret_cast<uint32_t*>(payload);
  const int n = a.n, H = a.H, nchunks = a.nchunks;
  constexpr int kSplit = pack_split<D>();
  const unsigned block = xcd_block(first);
  const unsigned bid = block >> parts.log2;
  const int sub = chunk_part(block, parts);
  const int seg = static_cast<int>(a.by_chunks.div(bid));  // (l * 2 + kv) * H + h
  const int chunk = static_cast<int>(bid) - seg * nchunks;
  const int lkv = static_cast<int>(a.by_heads.div(static_cast<uint32_t>(seg)));
  const int h = seg - lkv * H, kv = lkv & 1, l = lkv >> 1;
  const int g = group_of(a, l, h);
  const int t0 = chunk * kChunkTokens;
  const uint8_t* tier = a.tier + static_cast<size_t>(g) * n;
  const uint16_t* src = (kv ? a.v : a.k) + (static_cast<size_t>(l) * H + h) * static_cast<size_t>(n) * D;
  // the rows are loaded before the layout scan and the status check
  PackRows<D, pack_split<D>()> rows;
  pack_load(rows, src, tier, t0, n, sub);
  if (t0 + sub * (kChunkTokens / kSplit) >= n) return;  // no token of a short chunk in this part
  const uint32_t status = hdr[kGHdrStatus];
  {
    const int t = t0 + threadIdx.x;
    chunk_layout<D>(s, t < n ? tier[t] : kDROP,
                    reinterpret_cast<const uint32_t*>(payload + a.chunkidx_off +
                                                      static_cast<uint64_t>(g) * a.chunkidx_stride) +
                        2 * chunk);
  }
  if (status != 0u) return;  // a tier map is off its plan: nothing to pack
  __syncthreads();
  const uint64_t sc_off = a.segtab[2 * seg], row_off = a.segtab[2 * seg + 1];
  uint8_t* dst = payload + row_off;
  pack_store(s, rows, dst, reinterpret_cast<float*>(payload + sc_off), hdr + kGHdrNonfinite, sub);
  if (sub != 0) return;
  const uint32_t* e = a.group_table + 8 * g;
  if (chunk == nchunks - 1) {  // segment tail
    const uint64_t used = group_seg_bytes(e, D);
    const uint64_t stride = (used + 255u) / 256u * 256u;
    for (uint64_t b = used + 16ull * threadIdx.x; b < stride; b += 16ull * kRowThreads)
      st_nt16(dst + b, u32x4{0u, 0u, 0u, 0u});
  }
  if (chunk == 0 && kv == 1 && h == H - 1) {  // the layer's scale-section tail
    const uint64_t end = sc_off + 4ull * e[6];
    const uint64_t first_rows = a.segtab[2 * (l * 2 * H) + 1];
    zero_range(payload, end, first_rows, threadIdx.x, kRowThreads);
  }
}

__global__ void gunpack_init(const GroupArgs a) {
  if (threadIdx.x == 0) *a.status = 0u;
}

// grid: G + 1 workgroups.  Every metadata byte must be what the
// configuration, the group plans and the payload's own tier maps imply (the
// non-finite counter excepted); a failure sets the status to SKV_ERR_FORMAT.
__global__ __launch_bounds__(kMapThreads) void gunpack_check(const GroupArgs a) {
  __shared__ uint32_t s_chunk[kMaxChunks];
  __shared__ uint32_t s_bad;
  __shared__ CountScanLds s_scan;
  const uint8_t* __restrict__ payload = a.payload;
  const int tid = threadIdx.x;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  bool bad = false;
  if (blockIdx.x == static_cast<unsigned>(a.G)) {
    const uint32_t* hdr = reinterpret_cast<const uint32_t*>(payload);
    if (tid < 64 && tid != kGHdrNonfinite) bad |= hdr[tid] != gheader_word(a, tid);
    const uint32_t* gt = reinterpret_cast<const uint32_t*>(payload + a.group_off);
    for (int i = tid; i < 8 * a.G; i += kMapThreads) bad |= gt[i] != a.group_table[i];
    for (uint64_t b = a.group_off + 32ull * a.G + 4ull * tid; b < a.tiermaps_off; b += 4ull * kMapThreads)
      bad |= *reinterpret_cast<const uint32_t*>(payload + b) != 0u;
    const uint64_t* st = reinterpret_cast<const uint64_t*>(payload + a.segtab_off);
    const int nseg = 2 * a.L * a.H;
    for (int i = tid; i < 2 * nseg; i += kMapThreads) bad |= st[i] != a.segtab[i];
    for (uint64_t b = a.segtab_off + 16ull * nseg + 4ull * tid; b < a.layers_off; b += 4ull * kMapThreads)
      bad |= *reinterpret_cast<const uint32_t*>(payload + b) != 0u;
    const int nbt = (a.n + a.block_size - 1) / a.block_size;
    for (int i = tid; i < nbt; i += kMapThreads) {
      const int b = a.block_table[i];
      bad |= b < 0 || b >= a.num_blocks;
    }
    if (bad) atomicOr(&s_bad, 1u);
    __syncthreads();
    if (tid == 0 && s_bad) atomicOr(a.status, static_cast<uint32_t>(SKV_ERR_FORMAT));
    return;
  }
  const int g = blockIdx.x;
  const uint32_t* e = a.group_table + 8 * g;
  const int n = a.n, nchunks = a.nchunks;
  const int ngroups = (n + kGroupTokens - 1) / kGroupTokens;
  const uint64_t map_off = a.tiermaps_off + static_cast<uint64_t>(g) * a.tiermap_stride;
  const uint8_t* map = payload + map_off;
  for (int base = 0; base < ngroups; base += kMapBatch * kMapThreads) tally_map(map, n, ngroups, base, s_chunk);
  // codes of tokens >= n in the last word, and the map's padding, are zero
  if (tid == 0 && (n % kGroupTokens) != 0) {
    const uint32_t w = *reinterpret_cast<const uint32_t*>(map + 4ull * (ngroups - 1));
    bad |= (w >> (2 * (n % kGroupTokens))) != 0u;
  }
  for (uint64_t b = 4ull * ngroups + 4ull * tid; b < a.tiermap_stride; b += 4ull * kMapThreads)
    bad |= *reinterpret_cast<const uint32_t*>(map + b) != 0u;
  __syncthreads();
  // the chunk index equals the running sums; its padding is zero
  const int per = (nchunks + kMapThreads - 1) / kMapThreads;
  const int c0 = min(nchunks, tid * per), c1 = min(nchunks, c0 + per);
  const TierCounts mine = sum_chunks(s_chunk, c0, c1, bad);
  const CountScan sc = block_scan_counts(mine, false, s_scan);
  bad |= sc.total.n8 != e[2] || sc.total.n4 != e[3] || sc.total.nd != e[4];  // the FP16 count follows
  const uint64_t ci_off = a.chunkidx_off + static_cast<uint64_t>(g) * a.chunkidx_stride;
  TierCounts at = sc.before;
  for (int c = c0; c < c1; ++c) {
    const u32x2 w = reinterpret_cast<const u32x2*>(payload + ci_off)[c], want = index_entry(c, at);
    bad |= w.x != want.x || w.y != want.y;
    const TierCounts x = unpack_counts(s_chunk[c]);
    at.n8 += x.n8;
    at.n4 += x.n4;
    at.nd += x.nd;
  }
  for (uint64_t b = 8ull * nchunks + 4ull * tid; b < a.chunkidx_stride; b += 4ull * kMapThreads)
    bad |= *reinterpret_cast<const uint32_t*>(payload + ci_off + b) != 0u;
  if (bad) atomicOr(&s_bad, 1u);
  __syncthreads();
  if (tid == 0 && s_bad) atomicOr(a.status, static_cast<uint32_t>(SKV_ERR_FORMAT));
}

// grid: 2^parts.log2 workgroups (SPLIT, fewer where n is less than a chunk) for
// each of 2 * L * H * nchunks chunks, chunk fastest
template <int D, int SPLIT>
__global__ __launch_bounds__(kRowThreads) void gunpack_rows(const GroupArgs a, uint32_t first,
                                                            uint16_t* __restrict__ k_cache,
                                                            uint16_t* __restrict__ v_cache, ChunkParts parts) {
  __shared__ ChunkLds s;
  const uint32_t status = *a.status;
  const uint8_t* __restrict__ payload = a.payload;
  const int n = a.n, H = a.H, nchunks = a.nchunks, block_size = a.block_size;
  const bool short_segments = static_cast<unsigned>(nchunks) << parts.log2 <= kXcdRun;
  const unsigned block = short_segments ? xcd_block(first) : first + blockIdx.x;
  const unsigned bid = block >> parts.log2;
  const int sub = chunk_part(block, parts);
  const int seg = static_cast<int>(a.by_chunks.div(bid));
  const int chunk = static_cast<int>(bid) - seg * nchunks;
  const int lkv = static_cast<int>(a.by_heads.div(static_cast<uint32_t>(seg)));
  const int h = seg - lkv * H, kv = lkv & 1, l = lkv >> 1;
  const int g = group_of(a, l, h);
  const int t0 = chunk * kChunkTokens;
  if (t0 + sub * (kChunkTokens / SPLIT) >= n) return;  // no token of a short chunk in this part
  {
    const int t = t0 + threadIdx.x;
    int tr = kAbsent;
    uint32_t pos = 0;
    if (t < n) {
      const uint8_t* map = payload + a.tiermaps_off + static_cast<uint64_t>(g) * a.tiermap_stride;
      tr = (map[t >> 2] >> (2 * (t & 3))) & 3;
      const uint32_t block = a.by_block.div(static_cast<uint32_t>(t));
      pos = static_cast<uint32_t>(t) +
            (static_cast<uint32_t>(a.block_table[block]) - block) * static_cast<uint32_t>(block_size);
    }
    chunk_layout<D>(s, tr,
                    reinterpret_cast<const uint32_t*>(payload + a.chunkidx_off +
                                                      static_cast<uint64_t>(g) * a.chunkidx_stride) +
                        2 * chunk);
    if (status != 0u) return;  // payload rejected: write nothing
    if constexpr (SPLIT == 1) stage_scale(s, tr, reinterpret_cast<const float*>(payload + a.segtab[2 * seg]));
    s.pos[threadIdx.x] = pos;
  }
  __syncthreads();
  const uint8_t* src = payload + a.segtab[2 * seg + 1];
  uint16_t* cache = (kv ? v_cache : k_cache) + static_cast<size_t>(l) * a.num_blocks * block_size * H * D +
                    static_cast<size_t>(h) * D;
  unpack_chunk<D, SPLIT>(s, src, reinterpret_cast<const float*>(payload + a.segtab[2 * seg]), cache, H, sub);
}

GroupArgs group_args(const GroupLaunch& gl) {
  GroupArgs a{};
  a.group_table = gl.group_table;
  a.segtab = gl.segtab;
  a.L = gl.L;
  a.H = gl.H;
  a.d = gl.d;
  a.n = gl.n;
  a.gran = gl.gran;
  a.G = gl.G;
  a.nchunks = gl.nchunks;
  a.num_tiers = gl.num_tiers;
  a.score_mode = gl.score_mode;
  a.num_sink = gl.num_sink;
  a.budget_bits = gl.budget_bits;
  a.rho_bits = gl.rho_bits;
  a.decay_bits = gl.decay_bits;
  a.group_off = gl.group_off;
  a.tiermaps_off = gl.tiermaps_off;
  a.tiermap_stride = gl.tiermap_stride;
  a.chunkidx_off = gl.chunkidx_off;
  a.chunkidx_stride = gl.chunkidx_stride;
  a.segtab_off = gl.segtab_off;
  a.layers_off = gl.layers_off;
  a.total = gl.total;
  a.by_chunks = make_divider(static_cast<uint32_t>(gl.nchunks));
  a.by_heads = make_divider(static_cast<uint32_t>(gl.H));
  a.by_block = make_divider(1);
  return a;
}

}  // namespace

hipError_t launch_pack_groups(const GroupLaunch& gl, const uint16_t* k, const uint16_t* v, const uint8_t* tier,
                              uint8_t* payload, uint32_t* status, hipStream_t stream) {
  GroupArgs a = group_args(gl);
  a.k = k;
  a.v = v;
  a.tier = tier;
  a.payload = payload;
  a.status = status;
  gpack_init<<<1, 64, 0, stream>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  gpack_prep<<<a.G + 1, kMapThreads, 0, stream>>>(a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const uint64_t blocks = 2ull * a.L * a.H * static_cast<uint64_t>(a.nchunks);
#define SKV_GPACK(D)                                                                                    \
  {                                                                                                     \
    const ChunkParts parts = launch_parts<pack_split<D>()>(a.n, turned_parts(a.n));                     \
    e = launch_pieces(blocks << parts.log2, kRowThreads, [&](uint32_t first, uint32_t piece) {          \
      gpack_rows<D><<<piece, kRowThreads, 0, stream>>>(a, first, parts);                                \
    });                                                                                                 \
  }
  switch (a.d) {
    case 32: SKV_GPACK(32) break;
    case 64: SKV_GPACK(64) break;
    case 128: SKV_GPACK(128) break;
    case 256: SKV_GPACK(256) break;
    default: return hipErrorInvalidValue;
  }
#undef SKV_GPACK
  return e;
}

hipError_t launch_unpack_groups(const GroupLaunch& gl, const uint8_t* payload, uint16_t* k_cache, uint16_t* v_cache,
                                const int32_t* block_table, int32_t num_blocks, int32_t block_size,
                                uint32_t* status, hipStream_t stream) {
  GroupArgs a = group_args(gl);
  a.payload = const_cast<uint8_t*>(payload);
  a.status = status;
  a.block_table = block_table;
  a.num_blocks = num_blocks;
  a.block_size = block_size;
  a.by_block = make_divider(static_cast<uint32_t>(block_size));
  gunpack_init<<<1, 64, 0, stream>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  gunpack_check<<<a.G + 1, kMapThreads, 0, stream>>>(a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const uint64_t blocks = 2ull * a.L * a.H * static_cast<uint64_t>(a.nchunks);
#define SKV_GUNPACK_SPLIT(D, S)                                                                        \
  {                                                                                                    \
    ChunkParts parts = launch_parts<S>(a.n, turned_parts(a.n));                                        \
    parts.turned &= static_cast<uint32_t>(a.nchunks) << parts.log2 <= kXcdRun;                         \
    e = launch_pieces(blocks << parts.log2, kRowThreads, [&](uint32_t first, uint32_t piece) {         \
      gunpack_rows<D, S><<<piece, kRowThreads, 0, stream>>>(a, first, k_cache, v_cache, parts);        \
    });                                                                                                \
  }
#define SKV_GUNPACK(D)                                                           \
  if (blocks <= kTinyLaunch) SKV_GUNPACK_SPLIT(D, unpack_split_tiny<D>())        \
  else if (half_chunks<D>(a.n)) SKV_GUNPACK_SPLIT(D, unpack_split_half<D>())     \
  else if (blocks <= kShortLaunch) SKV_GUNPACK_SPLIT(D, unpack_split_short<D>()) \
  else SKV_GUNPACK_SPLIT(D, unpack_split_long<D>())
  switch (a.d) {
    case 32: SKV_GUNPACK(32) break;
    case 64: SKV_GUNPACK(64) break;
    case 128: SKV_GUNPACK(128) break;
    case 256: SKV_GUNPACK(256) break;
    default: return hipErrorInvalidValue;
  }
#undef SKV_GUNPACK
#undef SKV_GUNPACK_SPLIT
  return e;
}

}  // namespace skv
