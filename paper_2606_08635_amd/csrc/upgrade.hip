// Cold-tier precision upgrade (Sec. 4.2 and Fig. "sysarch": an on-demand fetch
// that upgrades tokens the decoder already holds at low precision; Sec. 8,
// "cold-tier fetch design").
//
// The prefill side, which still has the fp16 K/V and the tier map, packs for
// a list of tokens either their fp16 rows (FP16 mode: exact, 2 bytes per
// element) or the INT8 residual between each fp16 row and the row the
// decoder reconstructed (RESIDUAL8 mode: 1 byte per element plus a scale per
// row; the decoder's error drops to half a residual step).  The decoder
// applies the upgrade in place in its paged cache.
//   upg_prep   (one workgroup)  checks the token list, writes header, token
//                               list, tiers and padding;
//   upg_rows   (one workgroup per 8192 / d listed tokens of one (layer, K/V,
//                               head): UpgBlock) gathers the rows, recomputes
//                               the held row with the pack quantizer, quantizes
//                               the residual;
//   upg_check  (one workgroup)  checks an upgrade payload against the
//                               configuration and the block table;
//   upg_apply  (workgroups as upg_rows) adds the residual to (or overwrites)
//                               the cached rows.
#include <type_traits>

#include "device_util.h"
#include "row_codec.h"
#include "skv_internal.h"

namespace skv {
namespace {

constexpr int kUpgThreads = 256;  // threads of a row workgroup
constexpr int kUpgRows = 4;       // listed rows per thread, all loaded before any is processed
constexpr int kUpgCheckThreads = 1024;
constexpr uint32_t kUpgMagic = 0x55564B53u;  // "SKVU"
constexpr int kUpgHdrStatus = 18;

struct UpgArgs {
  const uint16_t* k;
  const uint16_t* v;
  const uint8_t* tier;
  const int32_t* tokens;  // pack: the caller's list
  uint8_t* up;            // the upgrade payload
  uint32_t* status;
  uint16_t* k_cache;
  uint16_t* v_cache;
  const int32_t* block_table;
  int32_t num_blocks, block_size;
  int32_t L, H, d, n, m, mode;
  uint64_t tokens_off, tiers_off, scales_off, data_off, total, row_bytes;
  Divider by_heads;  // by H
  Divider by_block;  // apply: by block_size
};

// The listed rows [i0, i0 + count) of one (layer, K or V, head) segment that a
// row workgroup handles.  Grid: x = ceil(m / count) workgroups, y and z = the
// segment, (layer * 2 + K or V) * H + head as in the payload, kUpgSegments to a z
// (a grid's y and z hold 16 bits), past the last one idle.  The order of the
// segments is the row kernels', so that a short request's apply finds the rows that
// unpack wrote in the same L2s (80 x 8 x 64, 126 of 130 tokens, residuals, unpack
// and apply: K and V of a pair side by side 36.1 us, so 27.2; 256
// rows per workgroup 30.3).
constexpr uint32_t kUpgSegments = 32768;

template <int D>
struct UpgBlock {
  static constexpr int kLanes = D / 8;                // lanes per row, 16 bytes each
  static constexpr int kStep = kUpgThreads / kLanes;  // rows the workgroup holds at a time
  static constexpr int kCount = kUpgRows * kStep;
  // Workgroups are dealt to XCDs in turn, so with few of them to a segment the last,
  // shorter ones of every list would all meet on the same XCDs: a hash of the
  // segment scatters where its workgroups begin.  80 x 8 pairs, d = 128, pack and
  // apply of 65 listed tokens, us: FP16 rows 15.7 -> 14.1 and 14.8 -> 12.9, residuals
  // 15.2 -> 14.6 and 19.6 -> 13.4 (256 rows per workgroup 15.4, 13.5, 24.9 and 15.1); of
  // 200 29.0 -> 28.3, 29.1 -> 27.8, 24.8 -> 24.0, 36.4 -> 33.2; from 8 workgroups on there
  // is nothing to gain.  At d = 32 two heads share a line of the cache, and residuals
  // of 800 tokens (four workgroups) lose it (40 -> 47), so only two are turned.
  static constexpr uint32_t kTurned = D == 32 ? 2 : 8;
  uint32_t kv, layer, head;
  uint32_t seg;
  int lane, row;  // the thread's 16 bytes of a row, its first listed row
  uint64_t seg_rows;  // the segment's first row in the payload
  __device__ __forceinline__ explicit UpgBlock(const UpgArgs& a) {
    seg = blockIdx.z * kUpgSegments + blockIdx.y;
    uint32_t x = blockIdx.x;
    if (gridDim.x <= kTurned) {
      x += __umulhi(seg * 0x9E3779B1u, gridDim.x);
      x -= x >= gridDim.x ? gridDim.x : 0u;
    }
    const uint32_t lkv = a.by_heads.div(seg);
    head = seg - lkv * a.H;
    kv = lkv & 1u;
    layer = lkv >> 1;
    lane = threadIdx.x % kLanes;
    row = static_cast<int>(x * kCount + threadIdx.x / kLanes);
    seg_rows = static_cast<uint64_t>(seg) * static_cast<uint64_t>(a.m);
  }
  __device__ __forceinline__ bool idle(const UpgArgs& a) const { return seg >= 2u * static_cast<uint32_t>(a.L * a.H); }
  static dim3 grid(const UpgArgs& a) {
    const uint32_t segments = 2u * static_cast<uint32_t>(a.L * a.H);
    return dim3(static_cast<uint32_t>((a.m + kCount - 1) / kCount), segments < kUpgSegments ? segments : kUpgSegments,
                (segments + kUpgSegments - 1) / kUpgSegments);
  }
};

__device__ __forceinline__ uint32_t upg_header_word(const UpgArgs& a, int i) {
  switch (i) {
    case 0: return kUpgMagic;
    case 1: return 1u;
    case 2: return static_cast<uint32_t>(a.L);
    case 3: return static_cast<uint32_t>(a.H);
    case 4: return static_cast<uint32_t>(a.d);
    case 5: return static_cast<uint32_t>(a.n);
    case 6: return static_cast<uint32_t>(a.m);
    case 7: return static_cast<uint32_t>(a.mode);
    case 8: return static_cast<uint32_t>(a.tokens_off);
    case 9: return static_cast<uint32_t>(a.tokens_off >> 32);
    case 10: return static_cast<uint32_t>(a.tiers_off);
    case 11: return static_cast<uint32_t>(a.tiers_off >> 32);
    case 12: return static_cast<uint32_t>(a.scales_off);
    case 13: return static_cast<uint32_t>(a.scales_off >> 32);
    case 14: return static_cast<uint32_t>(a.data_off);
    case 15: return static_cast<uint32_t>(a.data_off >> 32);
    case 16: return static_cast<uint32_t>(a.total);
    case 17: return static_cast<uint32_t>(a.total >> 32);
    default: return 0u;  // 18: status
  }
}

// The token list check shared by upg_prep and upg_check: every token in
// [0, n), strictly ascending, and (tier != null) its tier at most 3.  Loads are
// issued kListBatch at a time so the single workgroup keeps many in flight.
constexpr int kListBatch = 8;

__device__ __forceinline__ bool token_list_bad(const int32_t* tok, int m, int n, const uint8_t* tier_of_token,
                                               const uint8_t* tier_of_entry) {
  bool bad = false;
  for (int base = threadIdx.x; base < m; base += kListBatch * kUpgCheckThreads) {
    int t[kListBatch], prev[kListBatch];
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) {
      const int i = base + u * kUpgCheckThreads;
      t[u] = i < m ? tok[i] : 0;
      prev[u] = (i > 0 && i < m) ? tok[i - 1] : -1;
    }
    uint32_t tr[kListBatch];
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) {
      const int i = base + u * kUpgCheckThreads;
      const bool in = t[u] >= 0 && t[u] < n;
      bad |= !in || prev[u] >= t[u];
      tr[u] = 0;
      if (i < m && tier_of_token != nullptr && in) tr[u] = tier_of_token[t[u]];
      if (i < m && tier_of_entry != nullptr) tr[u] = tier_of_entry[i];
    }
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) bad |= tr[u] > 3u;
  }
  return bad;
}

__global__ __launch_bounds__(kUpgCheckThreads) void upg_prep(const UpgArgs a) {
  __shared__ uint32_t s_bad;
  const int tid = threadIdx.x;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  if (token_list_bad(a.tokens, a.m, a.n, a.tier, nullptr)) atomicOr(&s_bad, 1u);
  __syncthreads();
  const uint32_t status = s_bad ? static_cast<uint32_t>(SKV_ERR_INVALID_ARG) : 0u;
  uint8_t* up = a.up;
  if (tid < 64) reinterpret_cast<uint32_t*>(up)[tid] = tid == kUpgHdrStatus ? status : upg_header_word(a, tid);
  if (tid == 0 && a.status) *a.status = status;
  if (status) return;  // block-uniform
  int32_t* out_tok = reinterpret_cast<int32_t*>(up + a.tokens_off);
  uint8_t* out_tier = up + a.tiers_off;
  for (int base = tid; base < a.m; base += kListBatch * kUpgCheckThreads) {
    int t[kListBatch];
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) {
      const int i = base + u * kUpgCheckThreads;
      t[u] = i < a.m ? a.tokens[i] : 0;
    }
    uint8_t tr[kListBatch];
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) tr[u] = a.tier[t[u]];  // t in range: checked above
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) {
      const int i = base + u * kUpgCheckThreads;
      if (i < a.m) {
        out_tok[i] = t[u];
        out_tier[i] = tr[u];
      }
    }
  }
  for (uint64_t b = a.tokens_off + 4ull * a.m + tid; b < a.tiers_off; b += kUpgCheckThreads) up[b] = 0;
  for (uint64_t b = a.tiers_off + static_cast<uint64_t>(a.m) + tid; b < a.scales_off; b += kUpgCheckThreads) up[b] = 0;
  const uint64_t scales_end = a.scales_off + (a.mode == 1 ? 8ull * a.L * a.H * a.m : 0ull);
  for (uint64_t b = scales_end + tid; b < a.data_off; b += kUpgCheckThreads) up[b] = 0;
}

// INT8 codes of the lane's 8 residuals e (binary32) for a row whose largest
// magnitude is emax; zero gives codes 0.
__device__ __forceinline__ u32x2 residual_codes(const float (&e)[8], float emax, bool zero) {
  // RN32(127/a) for the binary32 residual maximum a without a division, and
  // no clamp: the sequence is correctly rounded and RN32(a RN32(127/a)) <
  // 127.5 for every binary32 a (checked exhaustively), so |e| <= a never codes
  // beyond +-127
  const float rcp = zero ? 0.0f : recip_scale_of_f32(emax, 127.0f);
  LaneCodes q;
#pragma unroll
  for (int i = 0; i < 8; ++i) q.c[i] = __builtin_bit_cast(uint32_t, e[i] * rcp + 12582912.0f);
  return pack_int8(q);
}

// The INT8 residual codes of one lane's 8 values against the held row, and the
// row's scale (all lanes of a row take part in the two row reductions).
// Neighbouring rows of a wave are held at different tiers, so nothing branches
// on the tier: a held code is RN(x RN32(Q / a)) with Q = 127 or 7, its value
// RN16(RN32(code RN32(a / Q))), and a reciprocal and a scale of 0 make the held
// row 0 (dropped rows, and rows of zeros).  A verbatim row has no residual; a
// row with an infinity or NaN, at whatever tier, has scale NaN and codes 0.
template <int LPR>
__device__ __forceinline__ u32x2 residual_lane(int tr, u32x4 x, float* scale) {
  const uint32_t amax = group_max<LPR>(absmax_bits8(x));
  const bool nonfinite = amax >= 0x7C00u;
  const bool held = (tr == kINT8 || tr == kINT4) && amax != 0u && !nonfinite;
  const float Qf = tr == kINT8 ? 127.0f : 7.0f;
  const float inv_q = tr == kINT8 ? 1.0f / 127.0f : 1.0f / 7.0f;  // RN32(1/Q)
  const float a = half_lo(amax);
  const float hs = held ? scale_of(a, Qf, inv_q) : 0.0f;
  const float hr = held ? recip_scale_of(a, Qf) : 0.0f;
  if (nonfinite) x = u32x4{0u, 0u, 0u, 0u};
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
  float e[8];
  float emax = 0.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float c0 = (half_mul<0>(w[j], hr) + 12582912.0f) - 12582912.0f;
    const float c1 = (half_mul<1>(w[j], hr) + 12582912.0f) - 12582912.0f;
    e[2 * j] = half_diff<0>(w[j], half_bits(scaled(c0, hs)));
    e[2 * j + 1] = half_diff<1>(w[j], half_bits(scaled(c1, hs)));
    emax = max_magnitude(e[2 * j], e[2 * j + 1], emax);
  }
  emax = __builtin_bit_cast(float, group_max<LPR>(__builtin_bit_cast(uint32_t, emax)));
  const bool zero = nonfinite || tr == kFP16 || emax == 0.0f;
  *scale = nonfinite ? __builtin_bit_cast(float, 0x7FC00000u) : zero ? 0.0f : scale_of(emax, 127.0f, 1.0f / 127.0f);
  return residual_codes(e, emax, zero);
}

// Both row kernels are bound by bytes in flight, the residual form also by
// vector instructions.  A workgroup takes one batch of rows (4 per thread, 16
// KiB of K or V) instead of four in turn, needs no shared memory and no
// barrier (a row's lanes read its token id and tier as one broadcast load),
// and holds at most 64 registers, so 8 waves stay on a SIMD: without that
// bound the compiler takes 72 and the pack 60 us where it now takes 48.  At
// 28 x 4 x 128, 3000 of 6000 tokens, pack and apply with their check launches
// (256 rows per workgroup before -> now): residuals 70 -> 48 and 85 -> 70 us,
// FP16 rows 73 -> 62 and 73 -> 67; 32 x 8 x 128, 16000 tokens, residuals 665 ->
// 552 (5.8 TB/s) and 1058 -> 1037; 4 x 4 x 128, 300 tokens, 18 -> 8 and 16 -> 7.
template <int D, int MODE>
__global__ __launch_bounds__(kUpgThreads, 8) void upg_rows(const UpgArgs a) {
  using B = UpgBlock<D>;
  const B b(a);
  if (b.idle(a)) return;
  uint8_t* up = a.up;
  const uint16_t* src = (b.kv ? a.v : a.k) +
                        static_cast<size_t>(b.layer * a.H + b.head) * static_cast<size_t>(a.n) * D + b.lane * 8;
  // The token ids are clamped into [0, n): the reads stay inside K/V and the
  // tier map even for a list the check refuses (then nothing is written), and
  // the clamp changes nothing for a valid list.
  int t[kUpgRows];
#pragma unroll
  for (int u = 0; u < kUpgRows; ++u) {
    const int i = b.row + u * B::kStep;
    t[u] = i < a.m ? min(max(a.tokens[i], 0), a.n - 1) : 0;
  }
  u32x4 x[kUpgRows];
  int tr[kUpgRows];
#pragma unroll
  for (int u = 0; u < kUpgRows; ++u) {
    x[u] = u32x4{0u, 0u, 0u, 0u};
    tr[u] = kDROP;
    if (b.row + u * B::kStep < a.m) {
      x[u] = ld_nt16(src + static_cast<size_t>(t[u]) * D);
      if constexpr (MODE == 1) tr[u] = a.tier[t[u]];
    }
  }
  if (reinterpret_cast<const uint32_t*>(up)[kUpgHdrStatus] != 0u) return;
#pragma unroll
  for (int u = 0; u < kUpgRows; ++u) {
    const int i = b.row + u * B::kStep;
    if constexpr (MODE == 0) {
      if (i < a.m) st_nt16(up + a.data_off + (b.seg_rows + i) * (2 * D) + b.lane * 16, x[u]);
    } else {
      float scale;
      const u32x2 codes = residual_lane<B::kLanes>(tr[u], x[u], &scale);
      if (i < a.m) {
        st_nt8(up + a.data_off + (b.seg_rows + i) * D + b.lane * 8, codes);
        if (b.lane == 0) reinterpret_cast<float*>(up + a.scales_off)[b.seg_rows + i] = scale;
      }
    }
  }
}

__global__ __launch_bounds__(kUpgCheckThreads) void upg_check(const UpgArgs a) {
  __shared__ uint32_t s_bad;
  const int tid = threadIdx.x;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  const uint8_t* up = a.up;
  if (tid <= kUpgHdrStatus && reinterpret_cast<const uint32_t*>(up)[tid] != upg_header_word(a, tid))
    atomicOr(&s_bad, 1u);
  __syncthreads();
  if (s_bad) {
    if (tid == 0) *a.status = static_cast<uint32_t>(SKV_ERR_FORMAT);
    return;
  }
  bool bad = token_list_bad(reinterpret_cast<const int32_t*>(up + a.tokens_off), a.m, a.n, nullptr,
                            up + a.tiers_off);
  const int nbt = (a.n + a.block_size - 1) / a.block_size;
  for (int base = tid; base < nbt; base += kListBatch * kUpgCheckThreads) {
    int b[kListBatch];
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) {
      const int i = base + u * kUpgCheckThreads;
      b[u] = i < nbt ? a.block_table[i] : 0;
    }
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) bad |= b[u] < 0 || b[u] >= a.num_blocks;
  }
  if (bad) atomicOr(&s_bad, 1u);
  __syncthreads();
  if (tid == 0) *a.status = s_bad ? static_cast<uint32_t>(SKV_ERR_FORMAT) : 0u;
}

// out = RN16(RN32(held + RN32(code * scale))) for the lane's 8 elements.
__device__ __forceinline__ u32x4 add_residual(u32x4 held, u32x2 c, float scale) {
  const uint32_t hs[4] = {held.x, held.y, held.z, held.w};
  const uint32_t cw[2] = {c.x, c.y};
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t w = cw[j >> 1];
    const int sh = 16 * (j & 1);
    const float c0 = static_cast<float>(static_cast<int32_t>(w << (24 - sh)) >> 24) * scale;
    const float c1 = static_cast<float>(static_cast<int32_t>(w << (16 - sh)) >> 24) * scale;
    o[j] = pack_half2(half_lo(hs[j]) + c0, half_hi(hs[j]) + c1);
  }
  const u32x4 out{o[0], o[1], o[2], o[3]};
  // only an infinite scale makes a NaN (code 0, or an infinity of the other
  // sign): written as 0x7E00
  return __builtin_isinf(scale) ? canon_nan_lane(out) : out;
}

template <int D, int MODE>
__global__ __launch_bounds__(kUpgThreads, 8) void upg_apply(const UpgArgs a) {
  using B = UpgBlock<D>;
  const B b(a);
  if (b.idle(a)) return;
  const uint8_t* up = a.up;
  // The payload's rows lie at fixed places inside it whatever its contents, and
  // the token ids are clamped into [0, n), so all of this may be read before the
  // check's verdict is known; the cache may not.
  u32x4 x[kUpgRows];
  u32x2 c[kUpgRows];
  float scale[kUpgRows];
  int t[kUpgRows];
#pragma unroll
  for (int u = 0; u < kUpgRows; ++u) {
    const int i = b.row + u * B::kStep;
    t[u] = 0;
    scale[u] = __builtin_bit_cast(float, 0x7FC00000u);
    if (i < a.m) {
      t[u] = min(max(reinterpret_cast<const int32_t*>(up + a.tokens_off)[i], 0), a.n - 1);
      if constexpr (MODE == 0) {
        x[u] = ld_nt16(up + a.data_off + (b.seg_rows + i) * (2 * D) + b.lane * 16);
      } else {
        scale[u] = reinterpret_cast<const float*>(up + a.scales_off)[b.seg_rows + i];
        c[u] = ld_nt8(up + a.data_off + (b.seg_rows + i) * D + b.lane * 8);
      }
    }
  }
  uint32_t pos[kUpgRows];
#pragma unroll
  for (int u = 0; u < kUpgRows; ++u) {
    const uint32_t blk = a.by_block.div(static_cast<uint32_t>(t[u]));
    pos[u] = static_cast<uint32_t>(a.block_table[blk]) * static_cast<uint32_t>(a.block_size) +
             (static_cast<uint32_t>(t[u]) - blk * static_cast<uint32_t>(a.block_size));
  }
  if (*a.status != 0u) return;
  uint16_t* cache = (b.kv ? a.v_cache : a.k_cache) +
                    static_cast<size_t>(b.layer) * a.num_blocks * a.block_size * a.H * D +
                    static_cast<size_t>(b.head) * D + b.lane * 8;
  if constexpr (MODE == 1) {
#pragma unroll
    for (int u = 0; u < kUpgRows; ++u)
      if (b.row + u * B::kStep < a.m)
        x[u] = *reinterpret_cast<const u32x4*>(cache + static_cast<size_t>(pos[u]) * a.H * D);
  }
#pragma unroll
  for (int u = 0; u < kUpgRows; ++u) {
    u32x4* dst = reinterpret_cast<u32x4*>(cache + static_cast<size_t>(pos[u]) * a.H * D);
    if constexpr (MODE == 0) {
      if (b.row + u * B::kStep < a.m) st_nt16(dst, x[u]);
    } else {
      // a NaN scale (also set for rows past m) keeps the held row
      if (!__builtin_isnan(scale[u])) *dst = add_residual(x[u], c[u], scale[u]);
    }
  }
}

inline uint64_t up256(uint64_t x) { return (x + 255u) / 256u * 256u; }

template <int MODE, typename F>
hipError_t dispatch_d(int d, F&& f) {
  switch (d) {
    case 32: return f(std::integral_constant<int, 32>{}, std::integral_constant<int, MODE>{});
    case 64: return f(std::integral_constant<int, 64>{}, std::integral_constant<int, MODE>{});
    case 128: return f(std::integral_constant<int, 128>{}, std::integral_constant<int, MODE>{});
    case 256: return f(std::integral_constant<int, 256>{}, std::integral_constant<int, MODE>{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

uint64_t upgrade_bytes(int32_t L, int32_t H, int32_t d, int32_t m, int32_t mode, uint64_t* offsets) {
  const uint64_t rows = 2ull * L * H * static_cast<uint64_t>(m);
  const uint64_t tokens_off = 256, tiers_off = tokens_off + up256(4ull * m);
  const uint64_t scales_off = tiers_off + up256(static_cast<uint64_t>(m));
  const uint64_t data_off = scales_off + (mode == 1 ? up256(rows * 4) : 0);
  const uint64_t row_bytes = mode == 0 ? 2ull * d : static_cast<uint64_t>(d);
  const uint64_t total = data_off + rows * row_bytes;
  if (offsets) {
    offsets[0] = tokens_off;
    offsets[1] = tiers_off;
    offsets[2] = scales_off;
    offsets[3] = data_off;
    offsets[4] = total;
    offsets[5] = row_bytes;
  }
  return total;
}

static UpgArgs upg_args(const Geometry& g, int32_t m, int32_t mode) {
  UpgArgs a{};
  a.L = g.L;
  a.H = g.H;
  a.d = g.d;
  a.n = g.n;
  a.m = m;
  a.mode = mode;
  a.by_heads = make_divider(static_cast<uint32_t>(g.H));
  uint64_t off[6];
  upgrade_bytes(g.L, g.H, g.d, m, mode, off);
  a.tokens_off = off[0];
  a.tiers_off = off[1];
  a.scales_off = off[2];
  a.data_off = off[3];
  a.total = off[4];
  a.row_bytes = off[5];
  return a;
}

hipError_t launch_pack_upgrade(const Geometry& g, const uint16_t* k, const uint16_t* v, const uint8_t* tier,
                               const int32_t* tokens, int32_t m, int32_t mode, uint8_t* out, uint32_t* status,
                               hipStream_t stream) {
  UpgArgs a = upg_args(g, m, mode);
  a.k = k;
  a.v = v;
  a.tier = tier;
  a.tokens = tokens;
  a.up = out;
  a.status = status;
  upg_prep<<<1, kUpgCheckThreads, 0, stream>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto run = [&](auto D, auto M) {
    upg_rows<decltype(D)::value, decltype(M)::value>
        <<<UpgBlock<decltype(D)::value>::grid(a), kUpgThreads, 0, stream>>>(a);
    return hipGetLastError();
  };
  return mode == 0 ? dispatch_d<0>(g.d, run) : dispatch_d<1>(g.d, run);
}

hipError_t launch_unpack_upgrade(const Geometry& g, const uint8_t* up, int32_t m, int32_t mode, uint16_t* k_cache,
                                 uint16_t* v_cache, const int32_t* block_table, int32_t num_blocks,
                                 int32_t block_size, uint32_t* status, hipStream_t stream) {
  UpgArgs a = upg_args(g, m, mode);
  a.up = const_cast<uint8_t*>(up);
  a.status = status;
  a.k_cache = k_cache;
  a.v_cache = v_cache;
  a.block_table = block_table;
  a.num_blocks = num_blocks;
  a.block_size = block_size;
  a.by_block = make_divider(static_cast<uint32_t>(block_size));
  upg_check<<<1, kUpgCheckThreads, 0, stream>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto run = [&](auto D, auto M) {
    upg_apply<decltype(D)::value, decltype(M)::value>
        <<<UpgBlock<decltype(D)::value>::grid(a), kUpgThreads, 0, stream>>>(a);
    return hipGetLastError();
  };
  return mode == 0 ? dispatch_d<0>(g.d, run) : dispatch_d<1>(g.d, run);
}

}  // namespace skv
