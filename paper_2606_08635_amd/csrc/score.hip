// Token scores (Sec. 4.3, eq. "importance"): KV-norm and recency modes.
//
// KV-norm mode ranks token t by I_t^2 = S_t * exp(-2 lambda (n-1-t)), where
// S_t is the sum of squares of every finite K and V element of the token over
// all layers and heads.  S_t is computed exactly, so the score is bit-exact
// whatever the reduction order:
//   * each binary16 x has x^2 a multiple of 2^-48 below 2^32; two FMAs split
//     it into a multiple of 2^-7 and a remainder of at most 2^-8 (acc_half);
//   * a thread adds at most 2^13 such terms into two binary64 accumulators,
//     which stay exact (multiples of 2^-7 below 2^46, and multiples of 2^-48
//     of at most 2^5);
//   * the accumulators become integers in units of 2^-48 and are combined in
//     128-bit integer arithmetic across lanes and layer groups.
// A non-finite input turns an accumulator into inf/NaN; only then does the
// thread redo its sum with non-finite elements skipped.
#include <algorithm>

#include "device_util.h"
#include "skv_internal.h"

namespace skv {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxPairsPerPart = 512;  // 2 tensors * 8 elements * 512 = 2^13 terms per thread
constexpr int kPairsInFlight = 2;  // pairs whose loads are issued together, parts of several pairs
#ifndef SKV_KVNORM_PAIR_INFLIGHT
#define SKV_KVNORM_PAIR_INFLIGHT 4  // row slices whose loads are issued together, one-pair parts
#endif
#ifndef SKV_KVNORM_PAIR_ROWS
#define SKV_KVNORM_PAIR_ROWS 8
#endif
constexpr int kPairRows = SKV_KVNORM_PAIR_ROWS;  // row slices per thread, one-pair parts

struct U128 {
  uint64_t lo, hi;
};

__device__ __forceinline__ U128 add128(U128 a, U128 b) {
  U128 r;
  r.lo = a.lo + b.lo;
  r.hi = a.hi + b.hi + (r.lo < a.lo ? 1u : 0u);
  return r;
}

// Correctly rounded (nearest-even) conversion of a 128-bit unsigned integer
// to binary64.
__device__ __forceinline__ double u128_to_double(U128 x) {
  if (x.hi == 0 && x.lo == 0) return 0.0;
  const int lz = x.hi ? __clzll(x.hi) : 64 + __clzll(x.lo);
  uint64_t top, rest;
  if (lz >= 64) {
    top = x.lo << (lz - 64);
    rest = 0;
  } else if (lz == 0) {
    top = x.hi;
    rest = x.lo;
  } else {
    top = (x.hi << lz) | (x.lo >> (64 - lz));
    rest = x.lo << lz;
  }
  uint64_t m = top >> 11;           // 53 significant bits
  const uint64_t rb = top & 0x7FFu;  // the 11 bits below them
  const bool up = rb > 0x400u || (rb == 0x400u && (rest != 0 || (m & 1u)));
  m += up ? 1u : 0u;
  return ldexp(static_cast<double>(m), 75 - lz);
}

// Adds the squares of the two halves of w to the exact sum kHiBase + sum = ah
// + al.  ah stays in [2^45, 2^46), where a binary64 moves in steps of 2^-7, so
// the first FMA adds x^2 rounded to a multiple of 2^-7, the difference of the
// two ah is exactly what was added, and the second FMA the exact remainder: a
// multiple of 2^-48 of at most 2^-8.
constexpr double kHiBase = 0x1p45;

__device__ __forceinline__ void acc_half(float f, double& ah, double& al) {
  const double x = static_cast<double>(f);
  const double s = __builtin_fma(x, x, ah);
  const double added = s - ah;
  ah = s;
  al += __builtin_fma(x, x, -added);
}

__device__ __forceinline__ void acc_word(uint32_t w, double& ah, double& al) {
  acc_half(half_lo(w), ah, al);
  acc_half(half_hi(w), ah, al);
}

__device__ __forceinline__ void acc_word_finite(uint32_t w, double& ah, double& al) {
  if (((w >> 10) & 31u) == 31u) w &= 0xFFFF0000u;
  if (((w >> 26) & 31u) == 31u) w &= 0x0000FFFFu;
  acc_word(w, ah, al);
}

__device__ __forceinline__ void acc16(u32x4 x, double& ah, double& al) {
  acc_word(x.x, ah, al);
  acc_word(x.y, ah, al);
  acc_word(x.z, ah, al);
  acc_word(x.w, ah, al);
}

__device__ __forceinline__ void acc16_finite(u32x4 x, double& ah, double& al) {
  acc_word_finite(x.x, ah, al);
  acc_word_finite(x.y, ah, al);
  acc_word_finite(x.z, ah, al);
  acc_word_finite(x.w, ah, al);
}

// The exact sum ah + al in units of 2^-48.  ah (without kHiBase) is a
// multiple of 2^-7 in [0, 2^45), al a multiple of 2^-48 in (-2^5, 2^5).
__device__ __forceinline__ U128 exact_units(double ah, double al) {
  const uint64_t a = static_cast<uint64_t>(ah * 0x1p7);
  const int64_t b = static_cast<int64_t>(al * 0x1p48);
  U128 s;
  s.lo = (a << 41) + static_cast<uint64_t>(b);
  s.hi = (a >> 23) + (s.lo < (a << 41) ? 1u : 0u) - (b < 0 ? 1u : 0u);
  return s;
}

// RN64 of a sum in units of 2^-48 (the scaling is exact: the sum is 0 or >= 2^-48)
__device__ __forceinline__ double units_to_double(U128 s) { return u128_to_double(s) * 0x1p-48; }

// One block: TOK tokens x all LPR lanes of their rows, over the (layer, head)
// pairs [part * pairs_per_part, (part + 1) * pairs_per_part): kPairsInFlight
// pairs (twice as many 16-byte loads) in flight per thread.  Writes the
// 128-bit partial sum of each token in units of 2^-48 to
// partial[(part * n + t) * 2 + {0: lo, 1: hi}] or, FINAL (the part is all that
// a score row sums), the score RN64(S) * w2[n-1-t] to score[part * n + t].
template <int D, bool FINAL>
__device__ __forceinline__ void kvnorm_partial_block(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                     int n, int pairs, int pairs_per_part,
                                                     uint64_t* __restrict__ partial, const double* __restrict__ w2,
                                                     double* __restrict__ score, int tok_block, int part) {
  constexpr int LPR = D / 8;
  constexpr int TOK = kThreads / LPR;
  constexpr int P = kPairsInFlight;
  __shared__ U128 s_part[kThreads];
  const int lane = threadIdx.x % LPR;
  const int r = threadIdx.x / LPR;
  const int t = tok_block * TOK + r;
  const int p0 = part * pairs_per_part;
  const int p1 = min(pairs, p0 + pairs_per_part);
  const size_t pair_stride = static_cast<size_t>(n) * D;  // elements between (l, h) pairs
  U128 sum{0, 0};
  if (t < n) {
    const size_t first = static_cast<size_t>(p0) * pair_stride + static_cast<size_t>(t) * D + lane * 8;
    const uint16_t* kp = k + first;
    const uint16_t* vp = v + first;
    double ah0 = kHiBase, al0 = 0.0, ah1 = kHiBase, al1 = 0.0;
    int p = p0;
    for (; p + P <= p1; p += P) {
      u32x4 a[P], b[P];
#pragma unroll
      for (int u = 0; u < P; ++u) {
        a[u] = ld_nt16(kp + u * pair_stride);
        b[u] = ld_nt16(vp + u * pair_stride);
      }
#pragma unroll
      for (int u = 0; u < P; ++u) {
        acc16(a[u], ah0, al0);
        acc16(b[u], ah1, al1);
      }
      kp += P * pair_stride;
      vp += P * pair_stride;
    }
    for (; p < p1; ++p) {
      const u32x4 a = ld_nt16(kp), b = ld_nt16(vp);
      acc16(a, ah0, al0);
      acc16(b, ah1, al1);
      kp += pair_stride;
      vp += pair_stride;
    }
    double ah = (ah0 - kHiBase) + (ah1 - kHiBase), al = al0 + al1;  // exact
    if (!(__builtin_isfinite(ah) && __builtin_isfinite(al))) {
      // an infinity or NaN was read: redo this thread's sum without them
      ah0 = kHiBase;
      al = 0.0;
      kp = k + first;
      vp = v + first;
      for (int q = p0; q < p1; ++q) {
        acc16_finite(ld_nt16(kp), ah0, al);
        acc16_finite(ld_nt16(vp), ah0, al);
        kp += pair_stride;
        vp += pair_stride;
      }
      ah = ah0 - kHiBase;
    }
    sum = exact_units(ah, al);
  }
  s_part[threadIdx.x] = sum;
  __syncthreads();
  if (lane == 0 && t < n) {
#pragma unroll
    for (int i = 1; i < LPR; ++i) sum = add128(sum, s_part[threadIdx.x + i]);
    const size_t idx = static_cast<size_t>(part) * n + t;
    if constexpr (FINAL) {
      score[idx] = units_to_double(sum) * w2[n - 1 - t];
    } else {
      partial[idx * 2] = sum.lo;
      partial[idx * 2 + 1] = sum.hi;
    }
  }
}

// grid: (token blocks, parts)
template <int D, bool FINAL>
__global__ __launch_bounds__(kThreads) void kvnorm_partial(const uint16_t* __restrict__ k,
                                                          const uint16_t* __restrict__ v, int n,
                                                          int pairs, int pairs_per_part,
                                                          uint64_t* __restrict__ partial,
                                                          const double* __restrict__ w2,
                                                          double* __restrict__ score) {
  kvnorm_partial_block<D, FINAL>(k, v, n, pairs, pairs_per_part, partial, w2, score, blockIdx.x, blockIdx.y);
}

// Every lane of each aligned group of G lanes (G = 4 .. 32) receives the sum
// of the group's binary64 values: butterfly steps by DPP lane moves inside
// 16-lane rows (each 64-bit value moved as two 32-bit halves), then one
// shuffle across the two rows of a 32-lane group.  The caller's values are
// integers in a common unit below 2^53 with their sum, so every order of
// addition gives the same exact result.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = dpp_mov<CTRL>(static_cast<uint32_t>(b));
  const uint32_t hi = dpp_mov<CTRL>(static_cast<uint32_t>(b >> 32));
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

template <int G>
__device__ __forceinline__ double group_sum_f64(double x) {
  static_assert(G == 4 || G == 8 || G == 16 || G == 32, "group size");
  x += dpp_f64<0xB1>(x);                          // quad_perm [1,0,3,2]
  x += dpp_f64<0x4E>(x);                          // quad_perm [2,3,0,1]
  if constexpr (G >= 8) x += dpp_f64<0x141>(x);   // row_half_mirror
  if constexpr (G >= 16) x += dpp_f64<0x140>(x);  // row_mirror
  if constexpr (G == 32) {  // lanes i and i ^ 16: lower + upper, the same sum in both (addition commutes)
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const LanePair lo = lane_pair16(static_cast<uint32_t>(b)), hi = lane_pair16(static_cast<uint32_t>(b >> 32));
    x = __builtin_bit_cast(double, (static_cast<uint64_t>(hi.lo) << 32) | lo.lo) +
        __builtin_bit_cast(double, (static_cast<uint64_t>(hi.hi) << 32) | lo.hi);
  }
  return x;
}

// Partial sums with one (layer, head) pair per part (per-head maps): block
// (x, y) covers pair y and the T * TOK consecutive tokens from x * T * TOK,
// i.e. one contiguous run of each of the pair's K and V planes.  A thread
// takes its T row slices S at a time, all 2 S loads issued before any is
// added (8 slices four at a time: 56 registers, 1 % faster than 4 slices two
// at a time; 4 slices four at a time or 8 eight at a time unroll into 114 or
// 502 registers and run far slower), and the lanes of a row combine their
// sums in binary64 by butterfly lane moves instead of through LDS.  That stays exact: a lane's
// sums hold 16 terms (8 K and 8 V elements), so over the LPR <= 32 lanes of
// a row the high parts, multiples of 2^-7, stay below 512 * 2^32 = 2^41 and
// the remainders, multiples of 2^-48, below 512 * 2^-8 = 2; both are exact,
// whatever the order.  A non-finite sum is redone from the registers
// without the non-finite elements.  The 128-bit sum is kvnorm_partial's.
// FINAL (each pair is a whole group): the block writes the group's score,
// RN64(S) * w2[n-1-t], into score[p * n + t], the value kvnorm_finish_groups
// would compute from the partial.
template <int D, int T, bool FINAL>
__global__ __launch_bounds__(kThreads) void kvnorm_partial_pairs(const uint16_t* __restrict__ k,
                                                                const uint16_t* __restrict__ v, int n,
                                                                uint64_t* __restrict__ partial,
                                                                const double* __restrict__ w2,
                                                                double* __restrict__ score) {
  constexpr int LPR = D / 8;
  constexpr int TOK = kThreads / LPR;
  const int lane = threadIdx.x % LPR;
  const int t0 = blockIdx.x * (T * TOK) + threadIdx.x / LPR;
  const int p = blockIdx.y;
  const size_t plane = static_cast<size_t>(p) * n * D;
  constexpr int S = SKV_KVNORM_PAIR_INFLIGHT < T ? SKV_KVNORM_PAIR_INFLIGHT : T;
  static_assert(T % S == 0, "whole groups of row slices");
#pragma unroll 1
  for (int i0 = 0; i0 < T; i0 += S) {  // S row slices (2 S 16-byte loads) in flight
    u32x4 kx[S], vx[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int t = t0 + (i0 + u) * TOK;
      kx[u] = u32x4{0u, 0u, 0u, 0u};
      vx[u] = u32x4{0u, 0u, 0u, 0u};
      if (t < n) {
        const size_t off = plane + static_cast<size_t>(t) * D + lane * 8;
        kx[u] = ld_nt16(k + off);
        vx[u] = ld_nt16(v + off);
      }
    }
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int t = t0 + (i0 + u) * TOK;
      double ah = kHiBase, al = 0.0;
      acc16(kx[u], ah, al);
      acc16(vx[u], ah, al);
      if (!(__builtin_isfinite(ah) && __builtin_isfinite(al))) {
        ah = kHiBase;
        al = 0.0;
        acc16_finite(kx[u], ah, al);
        acc16_finite(vx[u], ah, al);
      }
      ah = group_sum_f64<LPR>(ah - kHiBase);  // every lane of the row is active
      al = group_sum_f64<LPR>(al);
      if (lane == 0 && t < n) {
        const size_t idx = static_cast<size_t>(p) * n + t;
        if constexpr (FINAL) {
          // S = ah + al exactly, and one binary64 addition of the two exact
          // terms is the correctly rounded sum: RN64(S) without the 128-bit detour
          score[idx] = (ah + al) * w2[n - 1 - t];
        } else {
          const U128 sum = exact_units(ah, al);
          partial[idx * 2] = sum.lo;
          partial[idx * 2 + 1] = sum.hi;
        }
      }
    }
  }
}

// Request of a batched launch that owns flat block `b`: the last whose first
// block is at most b (one load, the starts across the wave's lanes).
__device__ __forceinline__ int score_request_of(const uint32_t (&begin)[kMaxScoreBatch], uint32_t b) {
  const int lane = threadIdx.x & 63;
  const uint32_t first = lane < kMaxScoreBatch ? begin[lane] : ~0u;
  return __popcll(__ballot(first <= b)) - 1;
}

// grid: (sum over requests of their token blocks, parts)
template <int D, bool FINAL>
__global__ __launch_bounds__(kThreads) void kvnorm_partial_batch(const ScoreBatchArgs a,
                                                                const double* __restrict__ w2) {
  const int req = score_request_of(a.tok_begin, blockIdx.x);
  const ScoreDesc& q = a.r[req];
  kvnorm_partial_block<D, FINAL>(q.k, q.v, q.n, a.pairs, a.pairs_per_part, q.partial, w2, q.score,
                                 static_cast<int>(blockIdx.x - a.tok_begin[req]), blockIdx.y);
}

// Sum of token t's partials of `parts` consecutive parts, eight in flight.
__device__ __forceinline__ U128 sum_parts(const uint64_t* __restrict__ partial, int parts, int n, int t) {
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  const u64x2* p = reinterpret_cast<const u64x2*>(partial) + t;
  U128 s{0, 0};
  int j = 0;
  for (; j + 8 <= parts; j += 8) {
    u64x2 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = p[static_cast<size_t>(j + u) * n];
#pragma unroll
    for (int u = 0; u < 8; ++u) s = add128(s, U128{x[u].x, x[u].y});
  }
  for (; j < parts; ++j) {
    const u64x2 x = p[static_cast<size_t>(j) * n];
    s = add128(s, U128{x.x, x.y});
  }
  return s;
}

__global__ __launch_bounds__(kThreads) void kvnorm_finish(const uint64_t* __restrict__ partial,
                                                         int parts, int n,
                                                         const double* __restrict__ w2,
                                                         double* __restrict__ score) {
  const int t = blockIdx.x * kThreads + threadIdx.x;
  if (t < n) score[t] = units_to_double(sum_parts(partial, parts, n, t)) * w2[n - 1 - t];
}

// grid: sum over requests of ceil(n / 256) blocks.  One decay table serves
// every request: entry Delta does not depend on n.
__global__ __launch_bounds__(kThreads) void kvnorm_finish_batch(const ScoreBatchArgs a, const double* __restrict__ w2) {
  const int req = score_request_of(a.fin_begin, blockIdx.x);
  const ScoreDesc& q = a.r[req];
  const int t = static_cast<int>(blockIdx.x - a.fin_begin[req]) * kThreads + threadIdx.x;
  if (t < q.n) q.score[t] = units_to_double(sum_parts(q.partial, a.parts, q.n, t)) * w2[q.n - 1 - t];
}

__global__ __launch_bounds__(kThreads) void recency_score_batch(const ScoreBatchArgs a, const double* __restrict__ w1) {
  const int req = score_request_of(a.fin_begin, blockIdx.x);
  const ScoreDesc& q = a.r[req];
  const int t = static_cast<int>(blockIdx.x - a.fin_begin[req]) * kThreads + threadIdx.x;
  if (t < q.n) q.score[t] = w1[q.n - 1 - t];
}

// grid: (token blocks, groups).  Group g's sum is the sum of its
// parts_per_group consecutive partials.
__global__ __launch_bounds__(kThreads) void kvnorm_finish_groups(const uint64_t* __restrict__ partial,
                                                                int parts_per_group, int n,
                                                                const double* __restrict__ w2,
                                                                double* __restrict__ score) {
  const int t = blockIdx.x * kThreads + threadIdx.x;
  if (t >= n) return;
  const uint64_t* p = partial + static_cast<size_t>(blockIdx.y) * parts_per_group * n * 2;
  score[static_cast<size_t>(blockIdx.y) * n + t] = units_to_double(sum_parts(p, parts_per_group, n, t)) * w2[n - 1 - t];
}

// grid: (token blocks, groups)
__global__ __launch_bounds__(kThreads) void recency_score_groups(const double* __restrict__ w1, int n,
                                                                double* __restrict__ score) {
  const int t = blockIdx.x * kThreads + threadIdx.x;
  if (t < n) score[static_cast<size_t>(blockIdx.y) * n + t] = w1[n - 1 - t];
}

__global__ __launch_bounds__(kThreads) void recency_score(const double* __restrict__ w1, int n,
                                                         double* __restrict__ score) {
  const int t = blockIdx.x * kThreads + threadIdx.x;
  if (t < n) score[t] = w1[n - 1 - t];
}

struct KvnormLaunch {
  int pairs, parts, pairs_per_part, blocks_tok;
};

// Parts of a row for about `blocks` workgroups: few enough pairs per part that
// each thread's binary64 sums stay exact.
KvnormLaunch kvnorm_split(const Geometry& g, int blocks) {
  KvnormLaunch s;
  s.pairs = g.L * g.H;
  const int tok = kThreads / (g.d / 8);
  s.blocks_tok = (g.n + tok - 1) / tok;
  int parts = (blocks + s.blocks_tok - 1) / s.blocks_tok;
  parts = max(parts, (s.pairs + kMaxPairsPerPart - 1) / kMaxPairsPerPart);
  parts = min(min(parts, s.pairs), 32768);  // a grid's y extent stays below 65536
  s.pairs_per_part = (s.pairs + parts - 1) / parts;
  s.parts = (s.pairs + s.pairs_per_part - 1) / s.pairs_per_part;
  return s;
}

// Parts of a row as a workspace reserves them: those of a launch of 65536
// workgroups.  Partial sums never need more.
KvnormLaunch kvnorm_reserved(const Geometry& g) { return kvnorm_split(g, 65536); }

// The launch is bound by HBM reads, so a part wants to be long enough that its
// loads outweigh its reduction and its 16-byte partials, and short enough that
// the workgroups in flight stay on few (layer, head) planes (one part over all
// 64 pairs of an 8 x 8 x 128 x 131072 request: 755 us, parts of 8 pairs 658).
// 8 pairs per part against one or two, as 65536 workgroups would give:
// 28 x 4 x 128 x 4096 85 -> 50 us (with the finish), 32 x 8 x 128 x 8189
// 242 -> 170 (6.3 TB/s), 4 x 4 x 64 x 262144 205 -> 171; from 32768 tokens of
// 32 x 8 x 128 on the reservation already gives 8.  Short launches, at most
// 4096 workgroups, take 4: 32 x 8 x 128 x 2048 56 -> 51 us, 28 x 4 x 128 x 700
// 18 -> 15.  One
// request of at most 768 workgroups of 4, three for each CU, takes 2, one round of
// loads: 1 x 8 x 64 x 2000 8.2 -> 6.9 us, 1 x 8 x 256 x 700 9.5 -> 8.3 (a batch of seven
// 1 x 8 x 32 x 2000 keeps 4: 6.6 us, with 2 7.4; up to 4 pairs one part has them all).
KvnormLaunch kvnorm_parts(const Geometry& g, bool one_request) {
  KvnormLaunch s = kvnorm_reserved(g);
  const int64_t blocks4 = static_cast<int64_t>(s.blocks_tok) * ((s.pairs + 3) / 4);
  const int64_t blocks8 = static_cast<int64_t>(s.blocks_tok) * ((s.pairs + 7) / 8);
  const int least = one_request && s.pairs > 4 && blocks4 <= 768 ? 2 : blocks8 <= 4096 ? 4 : 8;
  const int whole = (s.pairs_per_part + kPairsInFlight - 1) / kPairsInFlight * kPairsInFlight;
  s.pairs_per_part = min(max(least, whole), kMaxPairsPerPart);
  s.parts = (s.pairs + s.pairs_per_part - 1) / s.pairs_per_part;
  return s;
}

// Rows of one pair of more workgroups than this are streamed by
// kvnorm_partial_pairs, whose workgroups take eight times the tokens (with fewer
// they would be too few): 1 x 1 x 256 x 40000 16.1 -> 12.7 us, x 300000 93.8 -> 52.8
// (5.8 TB/s), 1 x 2 x 256 x 100000 45.7 -> 38.6, but 1 x 1 x 128 x 40000, 2500
// workgroups, 8.0 -> 8.9.
constexpr int kLongPair = 4800;

// One request: the parts above, but pairs_per_part 1 (kvnorm_partial_pairs) for
// long rows of one pair and, at d = 256, where a part's reduction is longest, of two.
KvnormLaunch kvnorm_shape(const Geometry& g) {
  KvnormLaunch s = kvnorm_parts(g, true);
  if (s.blocks_tok > kLongPair && (s.pairs == 1 || (s.pairs == 2 && g.d == 256 && kvnorm_reserved(g).parts == 2))) {
    s.pairs_per_part = 1;
    s.parts = s.pairs;
  }
  return s;
}

// Partials aligned to the groups of a granularity: a group's pairs are
// consecutive (pair p = l * H + h), so parts of pairs_per_part pairs never
// straddle two groups.
KvnormLaunch kvnorm_shape_groups(const Geometry& g, int gran, int* parts_per_group) {
  if (gran == SKV_GROUP_TOKEN) {
    const KvnormLaunch s = kvnorm_shape(g);
    *parts_per_group = s.parts;
    return s;
  }
  KvnormLaunch s;
  s.pairs = g.L * g.H;
  const int tok = kThreads / (g.d / 8);
  s.blocks_tok = (g.n + tok - 1) / tok;
  s.pairs_per_part = (gran == SKV_GROUP_LAYER && g.H <= kMaxPairsPerPart) ? g.H : 1;
  s.parts = s.pairs / s.pairs_per_part;
  *parts_per_group = gran == SKV_GROUP_LAYER ? g.H / s.pairs_per_part : 1;
  return s;
}

#define SKV_KVNORM_LAUNCH(KERNEL, GRID, FINAL, ...)                                        \
  switch (FINAL ? -g_d : g_d) {                                                             \
    case 32: KERNEL<32, false><<<GRID, kThreads, 0, stream>>>(__VA_ARGS__); break;          \
    case 64: KERNEL<64, false><<<GRID, kThreads, 0, stream>>>(__VA_ARGS__); break;          \
    case 128: KERNEL<128, false><<<GRID, kThreads, 0, stream>>>(__VA_ARGS__); break;        \
    case 256: KERNEL<256, false><<<GRID, kThreads, 0, stream>>>(__VA_ARGS__); break;        \
    case -32: KERNEL<32, true><<<GRID, kThreads, 0, stream>>>(__VA_ARGS__); break;          \
    case -64: KERNEL<64, true><<<GRID, kThreads, 0, stream>>>(__VA_ARGS__); break;          \
    case -128: KERNEL<128, true><<<GRID, kThreads, 0, stream>>>(__VA_ARGS__); break;        \
    case -256: KERNEL<256, true><<<GRID, kThreads, 0, stream>>>(__VA_ARGS__); break;        \
    default: return hipErrorInvalidValue;                                                   \
  }

// The partial-sum launch of shape s (FINAL: it writes the scores).
hipError_t launch_partial(const Geometry& g, const KvnormLaunch& s, bool final_scores, const uint16_t* k,
                          const uint16_t* v, const double* w2, uint64_t* partial, double* score, hipStream_t stream) {
  const dim3 grid(s.blocks_tok, s.parts);
  const int g_d = g.d;
  SKV_KVNORM_LAUNCH(kvnorm_partial, grid, final_scores, k, v, g.n, s.pairs, s.pairs_per_part, partial, w2, score)
  return hipGetLastError();
}

// One pair per part: each block streams a contiguous token run of one pair.
hipError_t launch_pairs(const Geometry& g, int pairs, bool final_scores, const uint16_t* k, const uint16_t* v,
                        const double* w2, uint64_t* partial, double* score, hipStream_t stream) {
#define SKV_PAIRS_LAUNCH(D)                                                                                      \
  {                                                                                                             \
    const dim3 pgrid((g.n + kPairRows * (kThreads / (D / 8)) - 1) / (kPairRows * (kThreads / (D / 8))), pairs);   \
    if (final_scores)                                                                                           \
      kvnorm_partial_pairs<D, kPairRows, true><<<pgrid, kThreads, 0, stream>>>(k, v, g.n, partial, w2, score);  \
    else                                                                                                        \
      kvnorm_partial_pairs<D, kPairRows, false><<<pgrid, kThreads, 0, stream>>>(k, v, g.n, partial, w2, score); \
  }
  switch (g.d) {
    case 32: SKV_PAIRS_LAUNCH(32); break;
    case 64: SKV_PAIRS_LAUNCH(64); break;
    case 128: SKV_PAIRS_LAUNCH(128); break;
    case 256: SKV_PAIRS_LAUNCH(256); break;
    default: return hipErrorInvalidValue;
  }
#undef SKV_PAIRS_LAUNCH
  return hipGetLastError();
}

}  // namespace

uint64_t kvnorm_scratch_bytes_groups(const Geometry& g, int32_t gran) {
  if (gran == SKV_GROUP_TOKEN) return kvnorm_scratch_bytes(g);
  int ppg;
  const KvnormLaunch s = kvnorm_shape_groups(g, gran, &ppg);
  if (s.pairs_per_part == 1 && ppg == 1) return 0;  // one pair per group: scores written directly
  return static_cast<uint64_t>(s.parts) * g.n * 16u;
}

hipError_t launch_score_kvnorm_groups(const Geometry& g, int32_t gran, int32_t G, const uint16_t* k,
                                      const uint16_t* v, const double* w2, uint64_t* partial, double* score,
                                      hipStream_t stream) {
  int ppg;
  const KvnormLaunch s = kvnorm_shape_groups(g, gran, &ppg);
  const bool final_scores = ppg == 1;  // a part is a whole group: the partial launch writes its scores
  if (s.pairs_per_part == 1) {
    const hipError_t e = launch_pairs(g, s.pairs, final_scores, k, v, w2, partial, score, stream);
    if (e != hipSuccess || final_scores) return e;
  } else {
    const hipError_t e = launch_partial(g, s, final_scores, k, v, w2, partial, score, stream);
    if (e != hipSuccess || final_scores) return e;
  }
  const dim3 fgrid((g.n + kThreads - 1) / kThreads, G);
  kvnorm_finish_groups<<<fgrid, kThreads, 0, stream>>>(partial, ppg, g.n, w2, score);
  return hipGetLastError();
}

hipError_t launch_score_recency_groups(const Geometry& g, int32_t G, const double* w1, double* score,
                                       hipStream_t stream) {
  const dim3 grid((g.n + kThreads - 1) / kThreads, G);
  recency_score_groups<<<grid, kThreads, 0, stream>>>(w1, g.n, score);
  return hipGetLastError();
}

uint64_t kvnorm_scratch_bytes(const Geometry& g) { return static_cast<uint64_t>(kvnorm_reserved(g).parts) * g.n * 16u; }

hipError_t launch_score_kvnorm(const Geometry& g, const uint16_t* k, const uint16_t* v,
                               const double* w2, uint64_t* partial, double* score,
                               hipStream_t stream) {
  const KvnormLaunch s = kvnorm_shape(g);
  const bool final_scores = s.parts == 1;
  const hipError_t e = s.pairs_per_part == 1
                           ? launch_pairs(g, s.pairs, final_scores, k, v, w2, partial, score, stream)
                           : launch_partial(g, s, final_scores, k, v, w2, partial, score, stream);
  if (e != hipSuccess || final_scores) return e;
  kvnorm_finish<<<(g.n + kThreads - 1) / kThreads, kThreads, 0, stream>>>(partial, s.parts, g.n, w2, score);
  return hipGetLastError();
}

void kvnorm_batch_shape(int32_t L, int32_t H, int32_t d, const int32_t* ns, int32_t count, ScoreBatchArgs* a) {
  uint64_t blocks = 0;
  const int tok = kThreads / (d / 8);
  for (int i = 0; i < count; ++i) blocks += (ns[i] + tok - 1) / tok;
  Geometry g{};
  g.L = L;
  g.H = H;
  g.d = d;
  // the single-request shape for a request as long as the whole batch: the
  // same number of workgroups per part, so the launch streams alike
  g.n = static_cast<int32_t>(std::min<uint64_t>(blocks * tok, kMaxTokens));
  const KvnormLaunch s = kvnorm_parts(g, false);
  a->pairs = s.pairs;
  a->pairs_per_part = s.pairs_per_part;
  a->parts = s.parts;
  a->reserved_parts = kvnorm_reserved(g).parts;
}

hipError_t launch_score_kvnorm_batch(const ScoreBatchArgs& a, int32_t d, const double* w2, hipStream_t stream) {
  const int tok = kThreads / (d / 8);
  uint32_t blocks = 0, fin = 0;
  for (int i = 0; i < a.count; ++i) {
    blocks += (a.r[i].n + tok - 1) / tok;
    fin += (a.r[i].n + kThreads - 1) / kThreads;
  }
  // rows of one pair, long on average: one launch each, as for one request
  if (a.pairs == 1 && blocks > static_cast<uint64_t>(kLongPair) * a.count) {
    for (int i = 0; i < a.count; ++i) {
      Geometry g{};
      g.d = d;
      g.n = a.r[i].n;
      const hipError_t e = launch_pairs(g, 1, true, a.r[i].k, a.r[i].v, w2, nullptr, a.r[i].score, stream);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const dim3 grid(blocks, a.parts);
  const int g_d = d;
  SKV_KVNORM_LAUNCH(kvnorm_partial_batch, grid, a.parts == 1, a, w2)
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.parts == 1) return e;
  kvnorm_finish_batch<<<fin, kThreads, 0, stream>>>(a, w2);
  return hipGetLastError();
}

hipError_t launch_score_recency_batch(const ScoreBatchArgs& a, const double* w1, hipStream_t stream) {
  uint32_t fin = 0;
  for (int i = 0; i < a.count; ++i) fin += (a.r[i].n + kThreads - 1) / kThreads;
  recency_score_batch<<<fin, kThreads, 0, stream>>>(a, w1);
  return hipGetLastError();
}

hipError_t launch_score_recency(const Geometry& g, const double* w1, double* score,
                                hipStream_t stream) {
  recency_score<<<(g.n + kThreads - 1) / kThreads, kThreads, 0, stream>>>(w1, g.n, score);
  return hipGetLastError();
}

}  // namespace skv
