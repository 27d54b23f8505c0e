// Quantize-and-pack (Algorithm 1, transfer; "standard symmetric" quantizer of
// Sec. 8), batched over requests of different lengths.
//
// pack_prep (one workgroup per request) checks the tier map against the plan,
// then writes the header, the 2-bit tier map and the chunk index; pack_rows
// (one to d/32 workgroups for each 256-token chunk of one (layer, K/V, head)
// segment of one request: pack_split, pack_split_variant and launch_parts in
// row_stream.h) rebuilds its chunk's row offsets with a block scan, reads each row
// with 16-byte loads (d/8 lanes per row), takes the row's absmax with a DPP
// lane reduction, quantizes in registers and stores the row at its offset.
// pack_keys (one workgroup per chunk) takes the K segments of a request with a
// per-channel tier.
// A launch may cover a range of layers: the payload is layer-major, so the
// layers of a request can be packed (and sent) in pieces.
#include "device_util.h"
#include "row_codec.h"
#include "row_stream.h"
#include "row_variants.h"
#include "skv_internal.h"
#include "tier_groups.h"

namespace skv {
namespace {

constexpr int kMaxChunks = kMaxTokens / kChunkTokens;

// grid: one workgroup per request.  Bound by latency: one round of loads, two
// barriers, one round of stores (rows past 131072 tokens take more rounds).
__global__ __launch_bounds__(kMapThreads) void pack_prep(const BatchArgs a) {
  __shared__ uint32_t s_chunk[kMaxChunks];
  __shared__ CountScanLds s_scan;
  const ReqDesc& r = a.r[blockIdx.x];
  const uint8_t* __restrict__ tier = r.tier;
  uint8_t* __restrict__ payload = r.payload;
  const int n = r.n, nchunks = r.nchunks;
  const int tid = threadIdx.x;
  const int ngroups = (n + kGroupTokens - 1) / kGroupTokens;
  const bool variant = (a.q8 | a.q4) != 0;  // launch-uniform

  // 1. counts per chunk; the map words of the first two batches stay in registers
  constexpr int kBatch = kMapBatch * kMapThreads;
  uint32_t map0[kMapBatch], map1[kMapBatch] = {};
  tally_tiers(tier, n, ngroups, 0, s_chunk, map0);
  if (ngroups > kBatch) tally_tiers(tier, n, ngroups, kBatch, s_chunk, map1);
  for (int base = 2 * kBatch; base < ngroups; base += kBatch) {
    uint32_t rest[kMapBatch];
    tally_tiers(tier, n, ngroups, base, s_chunk, rest);
  }
  uint32_t hword = 0u;  // the last wave has the least to do
  if (tid >= kMapThreads - 64) hword = header_word(a, r, tid & 63);
  __syncthreads();

  // 2. chunk starts: each thread owns a run of consecutive chunks
  const int per = (nchunks + kMapThreads - 1) / kMapThreads;
  const int c0 = min(nchunks, tid * per), c1 = min(nchunks, c0 + per);
  bool bad = false;
  const TierCounts mine = sum_chunks(s_chunk, c0, c1, bad);
  const CountScan sc = block_scan_counts(mine, bad, s_scan);
  const bool ok = !sc.bad && sc.total.n8 == static_cast<uint32_t>(r.n8) && sc.total.n4 == static_cast<uint32_t>(r.n4) &&
                  sc.total.nd == static_cast<uint32_t>(r.nd);  // the FP16 count follows
  const uint32_t status = ok ? 0u : static_cast<uint32_t>(SKV_ERR_INVALID_ARG);

  // 3. header (status recorded; the non-finite counter starts at zero)
  if (tid >= kMapThreads - 64)
    reinterpret_cast<uint32_t*>(payload)[tid & 63] = (tid & 63) == kHdrStatus ? status : hword;
  if (tid == 0 && r.status) *r.status = status;
  if (!ok) return;  // block-uniform

  // 4. chunk index
  TierCounts at = sc.before;
  for (int c = c0; c < c1; ++c) {
    const u32x2 e = index_entry(c, at);
    if (!variant) {
      reinterpret_cast<u32x2*>(payload + r.chunkidx_off)[c] = e;
    } else {  // 16-byte entries {units, quantized rows, V-side metadata bytes, K-side metadata bytes or 0}
      const bool chan = ((a.q8 | a.q4) & kQuantChannel) != 0;
      reinterpret_cast<u32x4*>(payload + r.chunkidx_off)[c] =
          u32x4{e.x, e.y, at.n8 * a.e8 + at.n4 * a.e4, chan ? at.n8 * a.ek8 + at.n4 * a.ek4 : 0u};
    }
    const TierCounts x = unpack_counts(s_chunk[c]);
    at.n8 += x.n8;
    at.n4 += x.n4;
    at.nd += x.nd;
  }
  zero_range(payload, r.chunkidx_off + (variant ? 16ull : 8ull) * nchunks, r.layers_off, tid, kMapThreads);

  // 5. the 2-bit tier map (4 bytes per group of 16 tokens), then its padding
  uint32_t* map = reinterpret_cast<uint32_t*>(payload + 256);
#pragma unroll
  for (int k = 0; k < kMapBatch; ++k) {
    const int g = k * kMapThreads + tid;
    if (g < ngroups) map[g] = map0[k];
    if (g + kBatch < ngroups) map[g + kBatch] = map1[k];
  }
  for (int g = 2 * kBatch + tid; g < ngroups; g += kMapThreads) {
    bool b;
    map[g] = map_from_tiers(load_tiers(tier, n, g), b);
  }
  zero_range(payload, 256 + 4ull * ngroups, r.chunkidx_off, tid, kMapThreads);
}

// Where a workgroup's rows go: the layer's block of the payload, the segment's
// rows and metadata.
struct PackDst {
  uint8_t *lay, *rows, *meta;
};
__device__ __forceinline__ PackDst pack_dst(const BatchArgs& a, const ReqDesc& r, const RowPlace& at) {
  uint8_t* lay = r.payload + r.layers_off + static_cast<uint64_t>(at.l) * r.layer_stride;
  return PackDst{lay,
                 lay + r.scales_bytes + r.channel_bytes + static_cast<uint64_t>(at.kv * a.H + at.h) * r.seg_stride,
                 lay + (at.kv == 0 ? static_cast<uint64_t>(at.h) * r.seg_scale_bytes_k
                                   : static_cast<uint64_t>(a.H) * r.seg_scale_bytes_k +
                                         static_cast<uint64_t>(at.h) * r.seg_scale_bytes)};
}

// Padding: the segment tail (last chunk), and the layer's per-row metadata tail
// and per-channel area tail.
template <int THREADS>
__device__ __forceinline__ void pack_padding(const BatchArgs& a, const ReqDesc& r, const RowPlace& at,
                                             const PackDst& d) {
  if (at.chunk == r.nchunks - 1) {
    for (uint64_t b = r.seg_bytes + 16ull * threadIdx.x; b < r.seg_stride; b += 16ull * THREADS)
      st_nt16(d.rows + b, u32x4{0u, 0u, 0u, 0u});
  }
  if (at.chunk == 0 && at.kv == 0 && at.h == 0) {
    // every metadata entry is 2, 4 or 8 bytes, so the used sizes are only
    // 2-byte aligned (the K and V halves differ with per-channel tiers):
    // 16-bit stores end exactly at each section boundary
    const uint64_t H = static_cast<uint64_t>(a.H);
    const uint64_t used = H * (r.seg_scale_bytes_k + r.seg_scale_bytes);
    for (uint64_t b = used + 2ull * threadIdx.x; b < r.scales_bytes; b += 2ull * THREADS)
      *reinterpret_cast<uint16_t*>(d.lay + b) = 0u;
    const uint64_t cused = H * static_cast<uint64_t>(r.nchunks) * (a.cb8 + a.cb4);
    for (uint64_t b = cused + 2ull * threadIdx.x; b < r.channel_bytes; b += 2ull * THREADS)
      *reinterpret_cast<uint16_t*>(d.lay + r.scales_bytes + b) = 0u;
  }
}

// grid: 2^parts.log2 workgroups (SPLIT, fewer where every request is shorter than
// a chunk) for each chunk of every segment of every request, or of the V segments
// only; a part of a chunk is always 256 / SPLIT tokens.  VARIANT: some tier uses a quantizer
// variant (row_variants.h); VALUES: the V segments only (the K segments have
// a per-channel tier and are pack_keys').
template <int D, int SPLIT, bool VARIANT, bool VALUES = false>
__global__ __launch_bounds__(kRowThreads) void pack_rows(const BatchArgs a, uint32_t first, ChunkParts parts) {
  __shared__ ChunkLds s;
  const uint32_t block = xcd_block(first);
  const uint32_t bid = block >> parts.log2;
  const int sub = chunk_part(block, parts);
  const int req = request_of_block(a, VALUES ? 2 * bid : bid);
  const ReqDesc& r = a.r[req];
  const uint32_t* hdr = reinterpret_cast<const uint32_t*>(r.payload);
  const int n = r.n;
  const RowPlace at = VALUES ? side_place(a, r, bid - a.begin[req] / 2, 1) : row_place(a, r, bid - a.begin[req]);
  const int chunk = at.chunk, kv = at.kv, t0 = chunk * kChunkTokens;
  const uint16_t* src = (kv ? r.v : r.k) + (static_cast<size_t>(at.l) * a.H + at.h) * static_cast<size_t>(n) * D;
  // the rows are loaded before the layout scan and the status check (the reads
  // stay inside K/V and the payload's metadata)
  PackRows<D, SPLIT> rows;
  pack_load(rows, src, r.tier, t0, n, sub);
  if (t0 + sub * (kChunkTokens / SPLIT) >= n) return;  // no token of a short chunk in this part
  const uint32_t status = hdr[kHdrStatus];

  // row offsets of this chunk: chunk-index base + block exclusive scan
  const VarCfg var{a.q8, a.q4, kv == 0 ? a.ek8 : a.e8, kv == 0 ? a.ek4 : a.e4};
  {
    const int t = t0 + threadIdx.x;
    const int tr = t < n ? r.tier[t] : kDROP;
    const uint32_t* cidx = reinterpret_cast<const uint32_t*>(r.payload + r.chunkidx_off);
    if constexpr (VARIANT) chunk_layout_var<D>(s, tr, cidx + 4 * chunk, 2, var);
    else chunk_layout<D>(s, tr, cidx + 2 * chunk);
  }
  if (status != 0u) return;  // tier map off plan: nothing to pack
  __syncthreads();

  const PackDst d = pack_dst(a, r, at);
  uint32_t* nonfinite = reinterpret_cast<uint32_t*>(r.payload) + kHdrNonfinite;
  if constexpr (VARIANT) pack_store_var(s, rows, d.rows, d.meta, nonfinite, var, sub);
  else pack_store(s, rows, d.rows, reinterpret_cast<float*>(d.meta), nonfinite, sub);
  if (sub == 0) pack_padding<kRowThreads>(a, r, at, d);
}

// grid: one workgroup for each chunk of every K segment of every request, with
// a per-channel tier: its K rows carry no per-row metadata (those of another
// tier, ROWS, do) and use the K-side metadata offsets of the chunk index.
template <int D, bool ROWS>
__global__ __launch_bounds__(KeyRows<D>::kThreads, 8) void pack_keys(const BatchArgs a, uint32_t first) {
  __shared__ ChunkLds s;
  __shared__ __align__(16) ChanLds<D> c;
  const uint32_t bid = first + blockIdx.x;
  const int req = request_of_block(a, 2 * bid);
  const ReqDesc& r = a.r[req];
  const uint32_t* hdr = reinterpret_cast<const uint32_t*>(r.payload);
  const int n = r.n;
  const RowPlace at = side_place(a, r, bid - a.begin[req] / 2, 0);
  const int t0 = at.chunk * kChunkTokens;
  KeyRows<D> rows;
  key_rows_load<D>(rows, r.k + (static_cast<size_t>(at.l) * a.H + at.h) * static_cast<size_t>(n) * D, r.tier, t0, n);
  chan_lds_init<D>(c);
  const uint32_t status = hdr[kHdrStatus];
  const VarCfg var{a.q8, a.q4, a.ek8, a.ek4};
  {
    const int t = t0 + threadIdx.x;
    const int tr = threadIdx.x < kChunkTokens && t < n ? r.tier[t] : kDROP;
    const uint32_t* cidx = reinterpret_cast<const uint32_t*>(r.payload + r.chunkidx_off);
    chunk_layout_var<D>(s, tr, cidx + 4 * at.chunk, 3, var);
  }
  if (status != 0u) return;  // tier map off plan: nothing to pack
  const PackDst d = pack_dst(a, r, at);
  uint8_t* blk = d.lay + r.scales_bytes + (static_cast<uint64_t>(at.h) * r.nchunks + at.chunk) * (a.cb8 + a.cb4);
  key_rows_store<D, ROWS>(s, c, rows, d.rows, d.meta, reinterpret_cast<uint32_t*>(r.payload) + kHdrNonfinite, var, blk,
                          blk + a.cb8);
  pack_padding<KeyRows<D>::kThreads>(a, r, at, d);
}

}  // namespace

hipError_t launch_pack(const BatchArgs& a, uint64_t rows, hipStream_t stream) {
  if (a.layer_begin == 0) {
    pack_prep<<<a.count, kMapThreads, 0, stream>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const bool variant = (a.q8 | a.q4) != 0;
  const bool chan = ((a.q8 | a.q4) & kQuantChannel) != 0;
  // some rows of a per-channel launch are quantized per row
  const bool mixed = (a.q8 & a.q4 & kQuantChannel) == 0;
  const int longest = longest_request(a);
  const bool turned = turned_parts(a);
  hipError_t e = hipSuccess;
#define SKV_PACK_ROWS(D, S, VARIANT, VALUES, CHUNKS)                                            \
  {                                                                                             \
    const ChunkParts parts = launch_parts<S>(longest, turned);                                  \
    e = launch_pieces((CHUNKS) << parts.log2, kRowThreads, [&](uint32_t first, uint32_t blocks) { \
      pack_rows<D, S, VARIANT, VALUES><<<blocks, kRowThreads, 0, stream>>>(a, first, parts);    \
    });                                                                                         \
  }
#define SKV_PACK_KEYS(D, ROWS)                                                                  \
  e = launch_pieces(rows / 2, KeyRows<D>::kThreads, [&](uint32_t first, uint32_t blocks) {      \
    pack_keys<D, ROWS><<<blocks, KeyRows<D>::kThreads, 0, stream>>>(a, first);                  \
  })
#define SKV_PACK_LAUNCH(D)                                                                      \
  if (!variant) {                                                                               \
    if (short_pack<D>(longest, rows)) SKV_PACK_ROWS(D, pack_split_short<D>(), false, false, rows) \
    else SKV_PACK_ROWS(D, pack_split<D>(), false, false, rows)                                  \
  } else if (!chan) {                                                                           \
    if (rows <= kShortLaunch) SKV_PACK_ROWS(D, pack_split<D>(), true, false, rows)              \
    else SKV_PACK_ROWS(D, pack_split_variant<D>(), true, false, rows)                           \
  } else {                                                                                      \
    if (mixed) SKV_PACK_KEYS(D, true);                                                          \
    else SKV_PACK_KEYS(D, false);                                                               \
    if (e != hipSuccess) return e;                                                              \
    if (rows <= kShortLaunch) SKV_PACK_ROWS(D, pack_split<D>(), true, true, rows / 2)           \
    else SKV_PACK_ROWS(D, pack_split_variant<D>(), true, true, rows / 2)                        \
  }
  switch (a.d) {
    case 32: SKV_PACK_LAUNCH(32) break;
    case 64: SKV_PACK_LAUNCH(64) break;
    case 128: SKV_PACK_LAUNCH(128) break;
    case 256: SKV_PACK_LAUNCH(256) break;
    default: return hipErrorInvalidValue;
  }
#undef SKV_PACK_LAUNCH
#undef SKV_PACK_KEYS
#undef SKV_PACK_ROWS
  return e;
}

}  // namespace skv
