// Decode-side dequantization into the fp16 paged cache (Sec. 4.2: only a
// lightweight per-tier dequantization runs after receipt).
//
// unpack_check (one workgroup per request) compares the payload header with
// the one the configuration implies, recounts the 2-bit tier map, re-derives
// the chunk index and range-checks the block table; it writes the verdict to
// the request's status word.  unpack_rows (one to four workgroups for each
// 256-token chunk of one (layer, K/V, head) segment of one request: the
// unpack_split functions and launch_parts in row_stream.h) writes nothing
// unless the verdict is 0; it rebuilds the chunk's row offsets with a block scan, loads
// each row at its tier's width, dequantizes in registers
// (RN16(RN32(code * scale))) and writes 16 bytes per lane into the token's
// paged slot.  Requests of a launch share the paged cache (each has its own
// block table); a launch may cover a range of layers.
#include "device_util.h"
#include "row_codec.h"
#include "row_stream.h"
#include "row_variants.h"
#include "skv_internal.h"
#include "tier_groups.h"

namespace skv {
namespace {

constexpr int kMaxChunks = kMaxTokens / kChunkTokens;

// grid: one workgroup per request.  Bound by latency: the header, the block
// table, the map and the chunk index load together (every address lies in the
// payload's metadata or the block table whatever their contents).
__global__ __launch_bounds__(kMapThreads) void unpack_check(const BatchArgs a, int num_blocks,
                                                            int block_size) {
  __shared__ uint32_t s_chunk[kMaxChunks];
  __shared__ uint32_t s_bad;
  __shared__ CountScanLds s_scan;
  const ReqDesc& r = a.r[blockIdx.x];
  const bool variant = (a.q8 | a.q4) != 0;  // launch-uniform
  const uint8_t* __restrict__ payload = r.payload;
  const int n = r.n, nchunks = r.nchunks;
  const int tid = threadIdx.x;
  const int nbt = (n + block_size - 1) / block_size;
  const int ngroups = (n + kGroupTokens - 1) / kGroupTokens;
  const uint32_t* cidx = reinterpret_cast<const uint32_t*>(payload + r.chunkidx_off);
  const int entry = variant ? 4 : 2;  // chunk-index words per chunk
  const int per = (nchunks + kMapThreads - 1) / kMapThreads;
  const int c0 = min(nchunks, tid * per), c1 = min(nchunks, c0 + per);
  if (tid == 0) s_bad = 0;
  bool bad = false;
  uint32_t hword = 0u;
  const int hi = tid - (kMapThreads - 64);  // header word of the last wave's lanes
  if (hi >= 0) hword = reinterpret_cast<const uint32_t*>(payload)[hi];
  uint32_t cidx_first[4] = {0u, 0u, 0u, 0u};
  if (c0 < c1) {
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (w < entry) cidx_first[w] = cidx[entry * c0 + w];
  }
  // block-table entries in range, eight loads in flight
  for (int base = 0; base < nbt; base += kMapBatch * kMapThreads) {  // block-uniform trip count
    int b[kMapBatch];
#pragma unroll
    for (int k = 0; k < kMapBatch; ++k) {
      const int i = base + k * kMapThreads + tid;
      b[k] = i < nbt ? r.block_table[i] : 0;
    }
#pragma unroll
    for (int k = 0; k < kMapBatch; ++k) bad |= b[k] < 0 || b[k] >= num_blocks;
  }
  // tier counts per chunk from the 2-bit map
  for (int base = 0; base < ngroups; base += kMapBatch * kMapThreads)
    tally_map(payload + 256, n, ngroups, base, s_chunk);
  // header: every word but the non-finite row counter must match
  if (hi >= 0 && hi != kHdrNonfinite) bad |= hword != header_word(a, r, hi);
  __syncthreads();
  const TierCounts mine = sum_chunks(s_chunk, c0, c1, bad);
  const CountScan sc = block_scan_counts(mine, false, s_scan);
  bad |= sc.total.n8 != static_cast<uint32_t>(r.n8) || sc.total.n4 != static_cast<uint32_t>(r.n4) ||
         sc.total.nd != static_cast<uint32_t>(r.nd);  // the FP16 count follows
  // the chunk index must equal the running sums
  TierCounts at = sc.before;
  for (int c = c0; c < c1; ++c) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = i >= entry ? 0u : c == c0 ? cidx_first[i] : cidx[entry * c + i];
    const u32x2 e = index_entry(c, at);
    bad |= w[0] != e.x || w[1] != e.y;
    if (variant) {
      const bool chan = ((a.q8 | a.q4) & kQuantChannel) != 0;
      bad |= w[2] != at.n8 * a.e8 + at.n4 * a.e4 || w[3] != (chan ? at.n8 * a.ek8 + at.n4 * a.ek4 : 0u);
    }
    const TierCounts x = unpack_counts(s_chunk[c]);
    at.n8 += x.n8;
    at.n4 += x.n4;
    at.nd += x.nd;
  }
  if (bad) atomicOr(&s_bad, 1u);
  __syncthreads();
  if (tid == 0) *r.status = s_bad ? static_cast<uint32_t>(SKV_ERR_FORMAT) : 0u;
}

// grid: sum over requests of nchunks * 2 * H * layer_count chunks, 2^parts.log2
// workgroups each (SPLIT, fewer where every request is shorter than a chunk; a
// part of a chunk is always 256 / SPLIT tokens).
// VARIANT: some tier uses a quantizer variant (row_variants.h); CHAN: some
// tier has per-channel keys (its own instantiation).
template <int D, bool VARIANT, bool CHAN = false, int SPLIT = 1>
__global__ __launch_bounds__(kRowThreads) void unpack_rows(const BatchArgs a, uint32_t first,
                                                           uint16_t* __restrict__ k_cache,
                                                           uint16_t* __restrict__ v_cache, int num_blocks,
                                                           int block_size, Divider by_block, bool short_segments,
                                                           ChunkParts parts) {
  __shared__ ChunkLds s;
  const uint32_t block = !VARIANT && short_segments ? xcd_block(first) : first + blockIdx.x;
  const uint32_t bid = block >> parts.log2;
  const int sub = chunk_part(block, parts);
  const int req = request_of_block(a, bid);
  const ReqDesc& r = a.r[req];
  const uint32_t status = *r.status;
  if constexpr (VARIANT)
    if (status != 0u) return;  // payload rejected: write nothing

  const uint8_t* __restrict__ payload = r.payload;
  const int n = r.n, H = a.H, nchunks = r.nchunks;
  const RowPlace at = row_place(a, r, bid - a.begin[req]);
  const int chunk = at.chunk, h = at.h, kv = at.kv, l = at.l;
  const int t0 = chunk * kChunkTokens;
  if (t0 + sub * (kChunkTokens / SPLIT) >= n) return;  // no token of a short chunk in this part
  // per-channel K tiers: K rows of those tiers decode with the chunk's channel
  // entries and use the K-side metadata offsets of the chunk index
  const bool chan_k = CHAN && kv == 0;
  const VarCfg var{a.q8, a.q4, kv == 0 ? a.ek8 : a.e8, kv == 0 ? a.ek4 : a.e4};
  {
    const int t = t0 + threadIdx.x;
    int tr = kAbsent;
    uint32_t pos = 0;
    if (t < n) {
      tr = (payload[256 + (t >> 2)] >> (2 * (t & 3))) & 3;
      const uint32_t block = by_block.div(static_cast<uint32_t>(t));
      pos = static_cast<uint32_t>(t) +
            (static_cast<uint32_t>(r.block_table[block]) - block) * static_cast<uint32_t>(block_size);
    }
    const uint32_t* cidx = reinterpret_cast<const uint32_t*>(payload + r.chunkidx_off);
    if constexpr (VARIANT) {
      chunk_layout_var<D>(s, tr, cidx + 4 * chunk, chan_k ? 3 : 2, var);
    } else {
      // the status is checked after the layout, so that its load is in flight
      // with the others (they stay inside the payload's metadata and the block
      // table whatever it says)
      chunk_layout<D>(s, tr, cidx + 2 * chunk);
      if (status != 0u) return;  // payload rejected: write nothing
      if constexpr (SPLIT == 1) {
        // the layer's scales of this segment (descriptor 0: one fp32 per quantized row)
        const uint8_t* lay0 = payload + r.layers_off + static_cast<uint64_t>(l) * r.layer_stride;
        stage_scale(s, tr, reinterpret_cast<const float*>(lay0 + static_cast<uint64_t>(kv * H + h) * r.seg_scale_bytes));
      }
    }
    s.pos[threadIdx.x] = pos;
  }
  __syncthreads();

  const uint8_t* lay = payload + r.layers_off + static_cast<uint64_t>(l) * r.layer_stride;
  const uint8_t* src = lay + r.scales_bytes + r.channel_bytes + static_cast<uint64_t>(kv * H + h) * r.seg_stride;
  const uint8_t* meta = lay + (kv == 0 ? static_cast<uint64_t>(h) * r.seg_scale_bytes_k
                                       : static_cast<uint64_t>(H) * r.seg_scale_bytes_k +
                                             static_cast<uint64_t>(h) * r.seg_scale_bytes);
  uint16_t* cache = (kv ? v_cache : k_cache) + static_cast<size_t>(l) * num_blocks * block_size * H * D +
                    static_cast<size_t>(h) * D;
  if constexpr (CHAN) {
    if (chan_k) {
      __shared__ ChanDecLds<D> c;
      const uint8_t* blk = lay + r.scales_bytes + (static_cast<uint64_t>(h) * nchunks + chunk) * (a.cb8 + a.cb4);
      const bool finite = load_channel_params<D>(c, blk, blk + a.cb8, var);
      unpack_chunk_var<D, true, SPLIT>(s, &c, finite, src, meta, cache, H, var, sub);
    } else {
      unpack_chunk_var<D, false, SPLIT>(s, nullptr, true, src, meta, cache, H, var, sub);
    }
  } else if constexpr (VARIANT) {
    unpack_chunk_var<D, false, SPLIT>(s, nullptr, true, src, meta, cache, H, var, sub);
  } else {
    unpack_chunk<D, SPLIT>(s, src, reinterpret_cast<const float*>(meta), cache, H, sub);
  }
}

}  // namespace

hipError_t launch_unpack(const BatchArgs& a, uint64_t rows, uint16_t* k_cache, uint16_t* v_cache,
                         int32_t num_blocks, int32_t block_size, hipStream_t stream) {
  if (a.layer_begin == 0) {
    unpack_check<<<a.count, kMapThreads, 0, stream>>>(a, num_blocks, block_size);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const bool variant = (a.q8 | a.q4) != 0;
  const bool chan = ((a.q8 | a.q4) & kQuantChannel) != 0;
  const Divider by_block = make_divider(static_cast<uint32_t>(block_size));
  const int longest = longest_request(a);
  const bool turned = turned_parts(a);
  const uint64_t segments = 2ull * a.count * a.H * a.layer_count;
  hipError_t e = hipSuccess;
#define SKV_UNPACK_SPLIT(D, V, C, S)                                                                \
  {                                                                                                 \
    ChunkParts parts = launch_parts<S>(longest, turned);                                            \
    const uint64_t total = rows << parts.log2;                                                      \
    const bool short_segments = total <= kXcdRun * segments;                                        \
    parts.turned &= short_segments;                                                                 \
    e = launch_pieces(total, kRowThreads, [&](uint32_t first, uint32_t blocks) {                    \
      unpack_rows<D, V, C, S><<<blocks, kRowThreads, 0, stream>>>(                                  \
          a, first, k_cache, v_cache, num_blocks, block_size, by_block, short_segments, parts);     \
    });                                                                                             \
  }
#define SKV_UNPACK_LAUNCH(D)                                                                        \
  if (!variant) {                                                                                  \
    if (rows <= kTinyLaunch) SKV_UNPACK_SPLIT(D, false, false, unpack_split_tiny<D>())             \
    else if (half_chunks<D>(longest)) SKV_UNPACK_SPLIT(D, false, false, unpack_split_half<D>())    \
    else if (rows <= kShortLaunch) SKV_UNPACK_SPLIT(D, false, false, unpack_split_short<D>())      \
    else SKV_UNPACK_SPLIT(D, false, false, unpack_split_long<D>())                                 \
  } else if (!chan) {                                                                              \
    if (rows <= kShortLaunch) SKV_UNPACK_SPLIT(D, true, false, unpack_split_short<D>())            \
    else SKV_UNPACK_SPLIT(D, true, false, unpack_split_variant<D>())                               \
  } else {                                                                                         \
    if (whole_chunks<D>(rows, segments)) SKV_UNPACK_SPLIT(D, true, true, 1)                        \
    else if (rows <= kShortLaunch) SKV_UNPACK_SPLIT(D, true, true, unpack_split_short<D>())        \
    else SKV_UNPACK_SPLIT(D, true, true, unpack_split_variant<D>())                                \
  }
  switch (a.d) {
    case 32: SKV_UNPACK_LAUNCH(32) break;
    case 64: SKV_UNPACK_LAUNCH(64) break;
    case 128: SKV_UNPACK_LAUNCH(128) break;
    case 256: SKV_UNPACK_LAUNCH(256) break;
    default: return hipErrorInvalidValue;
  }
#undef SKV_UNPACK_LAUNCH
#undef SKV_UNPACK_SPLIT
  return e;
}

}  // namespace skv
