// Tier assignment: sink pinning + importance-sorted cuts (Sec. 2.3 Prop. 1;
// Sec. 4.4; Algorithm 1, scoring and tier assignment).
//
// Non-sink token t carries the 64-bit ranking key
//   c_t = ((bits(score_t) >> 20) << 21) | t     (score <= 0 or NaN ranks as +0),
// all distinct.  With the tier counts fixed by the plan, token t gets FP16 iff
// c_t is among the n16 largest keys, INT8 iff among the next n8, INT4 iff
// among the next n4, DROP otherwise.  The kernel finds the three cut keys
// T1 >= T2 >= T3 (the n16-th, (n16+n8)-th and (n16+n8+n4)-th largest) by one
// radix select per cut over six digits (11, 11 and 10 bits of the key's high
// word, then the same of its low word), all three sharing each pass over the
// keys, then classifies every token against them.
//   * Resident form (at most 32768 non-sink tokens, one workgroup of 1024
//     threads): the scores are loaded once and the high words of the keys kept
//     in shared memory.  The first digit is not the exponent but the 11 leading
//     bits of the range that the row's keys span, which leaves a few dozen keys
//     in a cut's bin for most score distributions; a bin of at most 256 keys is
//     collected and ranked directly, and only fuller ones take further digits.
//   * Longer rows: the split form below when the caller gives scratch (one
//     launch per pass over the whole GPU; the same cuts), else one
//     workgroup that recomputes the keys from the scores on every pass (the
//     scores stay in L2), eight loads in flight per thread.  Both are done with
//     a cut once every key of its bin is admitted, mostly after two or three of
//     the six digits.
//   * Cuts with the same decided prefix share one histogram.
//   * Neighbouring tokens mostly share their leading digit (the decay orders
//     scores by position), so that pass must not serialize on one bin: a thread
//     counts the keys of consecutive tokens that fall in the same bin before
//     one atomic, and the lanes of a wave work on tokens far apart.
#include "device_util.h"
#include "skv_internal.h"

namespace skv {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kBins = 1 << 11;  // widest digit
constexpr int kPasses = 6;
constexpr int kBatch = 8;       // scores loaded per thread before they are counted
constexpr int kResident = 32;   // keys per thread held by the resident form
constexpr int kResidentSmall = 8;  // of its small instance: two workgroups per CU
constexpr int kList = 256;      // keys of a bin that are ranked directly

// Lowest key bit of digit `pass`: 53, 42, 32 in the high word, 21, 10, 0 in
// the low word.
__device__ __forceinline__ int digit_low_bit(int pass) {
  const int q = pass < 3 ? pass : pass - 3;
  return (pass < 3 ? 32 : 0) + (q == 2 ? 0 : 21 - 11 * q);
}

__device__ __forceinline__ uint64_t rank_key(double s, int t) {
  uint64_t bits = 0;
  if (s > 0.0) bits = __builtin_bit_cast(uint64_t, s);
  return ((bits >> 20) << 21) | static_cast<uint64_t>(static_cast<uint32_t>(t));
}

// Adds `count` keys to bin `bin` of histogram h unless count is zero.
__device__ __forceinline__ void flush(uint32_t* h, uint32_t bin, uint32_t count) {
  if (count) atomicAdd(&h[bin], count);
}

// One pass: histogram of the digit at `shift` over the keys whose decided
// bits equal the prefix of each active cut group.
struct RunCounter {
  uint32_t bin = 0, count = 0;
  __device__ __forceinline__ void add(uint32_t* h, uint32_t b) {
    if (b != bin) {
      flush(h, bin, count);
      bin = b;
      count = 0;
    }
    ++count;
  }
};

// Adds one to bin `bin` of h for every lane with `pred`: the lanes whose bin
// equals that of the first such lane by one atomic from that lane, the rest
// one atomic each.  Every active lane of the wave must call it.
__device__ __forceinline__ void wave_count(uint32_t* h, bool pred, uint32_t bin, int lane) {
  const uint64_t m = __ballot(pred);
  if (m == 0) return;  // wave-uniform
  const int leader = __ffsll(static_cast<unsigned long long>(m)) - 1;
  const uint32_t lb = static_cast<uint32_t>(__shfl(static_cast<int>(bin), leader));
  const uint64_t same = __ballot(pred && bin == lb);
  if (pred) {
    if (bin != lb)
      atomicAdd(&h[bin], 1u);
    else if (lane == leader)
      atomicAdd(&h[lb], static_cast<uint32_t>(__popcll(same)));
  }
}

// LDS state of one row's selection.
struct SelectState {
  uint32_t hist[3][kBins];
  uint64_t prefix[3];  // decided key bits of each cut
  uint32_t rank[3];    // remaining rank (1-based) inside the current prefix; 0: the cut is final
  int group[3];        // which histogram a cut reads
};

// After a pass's histograms are complete: wave j walks cut j's histogram
// from the top bin down and fixes the digit (at key bit `shift`) of the bin
// that holds its remaining rank (32 bins per lane).  A cut that admits every
// key of that bin is final whatever the bits below: its key is the bin's lowest,
// the prefix itself, and its rank becomes 0.
__device__ __forceinline__ void choose_digits(SelectState& st, int shift, int lane, int wave) {
  if (wave >= 3 || st.rank[wave] == 0) return;
  const int j = wave;
  constexpr int kPer = kBins / 64;  // 32 consecutive bins per lane, read 4 at a time
  const u32x4* h4 = reinterpret_cast<const u32x4*>(st.hist[st.group[j]]);
  const int b0 = kBins - kPer * (lane + 1);  // this lane's lowest bin; lane 0 holds the top
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < kPer / 4; ++i) {  // rotated by lane: lanes 128 B apart would share banks
    const u32x4 c = h4[b0 / 4 + ((i + lane) & (kPer / 4 - 1))];
    sum += c.x + c.y + c.z + c.w;
  }
  uint32_t inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = static_cast<uint32_t>(__shfl_up(static_cast<int>(inc), o));
    if (lane >= o) inc += y;
  }
  uint32_t run = inc - sum;  // keys in the bins above this lane's
  const uint32_t want = st.rank[j];
  if (run < want && want <= run + sum) {
    const uint64_t prefix = st.prefix[j];
#pragma unroll
    for (int i = kPer / 4 - 1; i >= 0; --i) {  // descending bins
      const u32x4 c = h4[b0 / 4 + i];
      const uint32_t cs[4] = {c.w, c.z, c.y, c.x};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int b = b0 + 4 * i + (3 - e);
        if (run < want && want <= run + cs[e]) {
          st.prefix[j] = prefix | (static_cast<uint64_t>(b) << shift);
          st.rank[j] = want - run == cs[e] ? 0u : want - run;
        }
        run += cs[e];
      }
    }
  }
}

// The key's high word (its low word holds 11 more score bits and the token).
__device__ __forceinline__ uint32_t rank_key_hi(double s) {
  return s > 0.0 ? static_cast<uint32_t>(__builtin_bit_cast(uint64_t, s) >> 31) : 0u;
}

__device__ __forceinline__ uint32_t uniform32(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(x)));
}
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  return static_cast<uint64_t>(uniform32(static_cast<uint32_t>(x >> 32))) << 32 | uniform32(static_cast<uint32_t>(x));
}

// Cut j reads the histogram of the first cut (in cut order) with a nonzero
// rank and the same decided prefix.
__device__ __forceinline__ int cut_group(const uint64_t (&prefix)[3], const uint32_t (&rank)[3], int j) {
  for (int i = 0; i < j; ++i)
    if (rank[i] != 0 && prefix[i] == prefix[j]) return i;
  return j;
}

// Shared state of the resident form.  A histogram's space also holds the list
// of its bin's keys.
struct ResidentState {
  uint32_t hist[3][kBins];
  uint64_t prefix[3];  // decided key bits (key >> pos) of each cut
  uint64_t cut[3];     // the cut keys
  uint32_t rank[3];    // remaining rank (1-based) inside the bin
  uint32_t count[3];   // keys of the bin
  uint32_t listed[3];  // keys collected so far, per histogram
  uint32_t lo[kSelThreads / 64], hi[kSelThreads / 64];  // per wave: smallest and largest high word
};
static_assert(kList * sizeof(uint64_t) <= kBins * sizeof(uint32_t), "a list fits its histogram");

// One wave: the bin of h that holds rank st.rank[j], counted from the top bin.
// Each lane sums 32 consecutive bins, then the lanes read the bins of the lane
// that holds the rank.
__device__ __forceinline__ uint32_t choose_bin(ResidentState& st, const uint32_t* h, int j, int lane) {
  constexpr int kPer = kBins / 64;
  const u32x4* h4 = reinterpret_cast<const u32x4*>(h);
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < kPer / 4; ++i) {  // rotated by lane: lanes 128 B apart would share banks
    const u32x4 c = h4[lane * (kPer / 4) + ((i + lane) & (kPer / 4 - 1))];
    sum += c.x + c.y + c.z + c.w;
  }
  const uint32_t want = st.rank[j];
  uint32_t inc = wave_inclusive_scan(sum);
  uint32_t above = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), 63)) - inc;
  const uint64_t at = __ballot(above < want && want <= above + sum);
  const int owner = __ffsll(static_cast<unsigned long long>(at)) - 1;
  const uint32_t base = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(above), owner));
  const uint32_t total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sum), owner));
  const uint32_t c = lane < kPer ? h[owner * kPer + lane] : 0u;
  inc = wave_inclusive_scan(c);
  above = base + total - inc;
  const bool mine = above < want && want <= above + c;
  const int bin = __ffsll(static_cast<unsigned long long>(__ballot(mine))) - 1;
  if (mine) {
    st.rank[j] = want - above;
    st.count[j] = c;
  }
  return static_cast<uint32_t>(owner * kPer + bin);
}

// Assignment of one score row of at most RES * 1024 non-sink tokens by one
// 1024-thread workgroup: load, histogram, bin choice, collection and ranking,
// five barriers where every cut's bin holds at most kList keys.  Bound by
// latency (at 32768 tokens also by shared-memory reads and atomics of the one
// CU).  Against six fixed digits, each with its histograms and a serial walk
// of 32 bins, at decayed KV-norm scores: 512 tokens 22 -> 4.7 us, 4096 26 ->
// 7.3, 8189 36 -> 12, 32768 58 -> 25; 336 rows of 4096 tokens, now two
// workgroups per CU, 57 -> 12.
template <int RES>
__device__ __forceinline__ void assign_resident(const double* __restrict__ score, uint8_t* __restrict__ tier, int n,
                                                int n_sink, int n16, int n8, int n4) {
  __shared__ __attribute__((aligned(16))) ResidentState st;
  __shared__ uint32_t hi[RES * kSelThreads];  // high word of non-sink token n_sink + i at hi[i]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = n - n_sink;
  const uint32_t cut_rank[3] = {static_cast<uint32_t>(n16), static_cast<uint32_t>(n16 + n8),
                                static_cast<uint32_t>(n16 + n8 + n4)};
  // a cut of rank 0 admits no key, one of rank m every key: nothing to select
  bool active[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) active[j] = cut_rank[j] != 0 && cut_rank[j] < static_cast<uint32_t>(m);

  uint32_t mn = ~0u, mx = 0u;
  {
    double sc[RES];
#pragma unroll
    for (int u = 0; u < RES; ++u)
      if (u * kSelThreads < m) sc[u] = score[min(n_sink + u * kSelThreads + tid, n - 1)];  // uniform condition
#pragma unroll
    for (int u = 0; u < RES; ++u) {
      const int i = u * kSelThreads + tid;
      if (i < m) {
        const uint32_t w = rank_key_hi(sc[u]);
        hi[i] = w;
        mn = min(mn, w);
        mx = max(mx, w);
      }
    }
  }
  for (int i = tid; i < kBins; i += kSelThreads) st.hist[0][i] = 0;
  if (tid < 3) {
    st.rank[tid] = tid == 0 ? cut_rank[0] : tid == 1 ? cut_rank[1] : cut_rank[2];
    st.count[tid] = 0;
    st.listed[tid] = 0;
    st.prefix[tid] = 0;
    st.cut[tid] = 0;
  }
  mx = wave_max(mx);
  mn = ~wave_max(~mn);
  if (lane == 0) {
    st.lo[wave] = mn;
    st.hi[wave] = mx;
  }
  __syncthreads();

  if (active[0] || active[1] || active[2]) {  // uniform
    mx = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(group_max<16>(st.hi[lane & 15]))));
    mn = ~static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(group_max<16>(~st.lo[lane & 15]))));
    // first digit: the keys' high words from bit `shift` up, counted from the smallest
    int shift = max(0, 32 - 11 - (mx == mn ? 32 : __builtin_clz(mx - mn)));
    if ((mx >> shift) - (mn >> shift) >= static_cast<uint32_t>(kBins)) ++shift;
    const uint32_t first_bin = mn >> shift;
    const int per = ((m + kSelThreads - 1) / kSelThreads) | 1;  // consecutive keys per thread; odd: no bank conflicts
    const int i0 = tid * per, i1 = min(m, i0 + per);
    {
      RunCounter r;
      for (int i = i0; i < i1; ++i) r.add(st.hist[0], (hi[i] >> shift) - first_bin);
      flush(st.hist[0], r.bin, r.count);
    }
    __syncthreads();
    if (wave < 3 && active[wave == 0 ? 0 : wave == 1 ? 1 : 2]) {
      const uint32_t bin = choose_bin(st, st.hist[0], wave, lane);
      if (lane == 0) st.prefix[wave] = first_bin + bin;
    }
    __syncthreads();
    int pos = 32 + shift;  // key bits below pos are undecided
    uint64_t pre[3];
    uint32_t rk[3];
    bool lead[3];     // the cut owns its histogram
    int hs;           // a key of cut j's bin has high word >> hs == hp[j]
    uint32_t hp[3];
    auto read_state = [&]() {  // all of it wave-uniform
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        pre[j] = uniform64(st.prefix[j]);
        rk[j] = active[j] ? uniform32(st.rank[j]) : 0u;
      }
      hs = max(0, pos - 32);
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        lead[j] = rk[j] != 0 && cut_group(pre, rk, j) == j;
        hp[j] = static_cast<uint32_t>(pos >= 32 ? pre[j] : pre[j] >> (32 - pos));
      }
    };
    auto in_bin = [&](uint32_t w) {  // of any cut, as far as the high word tells
      return (lead[0] && w >> hs == hp[0]) || (lead[1] && w >> hs == hp[1]) || (lead[2] && w >> hs == hp[2]);
    };
    read_state();
    const int token_bits = 32 - __builtin_clz(static_cast<uint32_t>(n - 1) | 1u);
    // fuller bins: further digits of at most 11 bits, down to the low word
    while (st.count[0] > kList || st.count[1] > kList || st.count[2] > kList) {  // uniform
      // pos falls to 32, 21 (the score's bits of the low word), the token's leading
      // 11 bits (of its 21 those past the row's length are zero, so of 65536
      // tokens at most 32 are left in a bin) and 0, where every key is alone
      const int next = pos > 32 ? max(32, pos - 11) : pos == 32 ? 21 : pos == 21 ? max(0, token_bits - 11) : 0;
      const uint32_t mask = (1u << (pos - next)) - 1u;
      for (int i = tid; i < 3 * kBins; i += kSelThreads) (&st.hist[0][0])[i] = 0;
      __syncthreads();
      RunCounter r0, r1, r2;
      if (pos > 32) {
        for (int i = i0; i < i1; ++i) {
          const uint32_t w = hi[i], d = w >> hs, bin = (w >> (next - 32)) & mask;
          if (lead[0] && d == hp[0]) r0.add(st.hist[0], bin);
          if (lead[1] && d == hp[1]) r1.add(st.hist[1], bin);
          if (lead[2] && d == hp[2]) r2.add(st.hist[2], bin);
        }
      } else {
        // The high word is decided, and the low word needs the scores again: a
        // wave takes consecutive keys, so that its loads are contiguous (kLow of
        // them in flight) and a lane's runs of equal bins still long.  With the
        // runs of consecutive keys that the threads count above, one load after
        // another, and the last digit of the token always taken: 32768 scores of
        // four values 96 us, so 79; sorted ones of 32 values 64 and 50.
        constexpr int kLow = RES <= kResidentSmall ? 4 : 8;
        const int rounds = (m + kSelThreads - 1) / kSelThreads, w0 = wave * 64 * rounds + lane;
        for (int b = 0; b < rounds; b += kLow) {
          double sc[kLow];
          bool in[kLow];
#pragma unroll
          for (int u = 0; u < kLow; ++u) {
            const int i = w0 + (b + u) * 64;
            in[u] = b + u < rounds && i < m && in_bin(hi[min(i, m - 1)]);
            sc[u] = in[u] ? score[n_sink + i] : 0.0;
          }
#pragma unroll
          for (int u = 0; u < kLow; ++u) {
            if (!in[u]) continue;
            const uint64_t key = rank_key(sc[u], n_sink + w0 + (b + u) * 64), d = key >> pos;
            const uint32_t bin = (static_cast<uint32_t>(key) >> next) & mask;
            if (lead[0] && d == pre[0]) r0.add(st.hist[0], bin);
            if (lead[1] && d == pre[1]) r1.add(st.hist[1], bin);
            if (lead[2] && d == pre[2]) r2.add(st.hist[2], bin);
          }
        }
      }
      flush(st.hist[0], r0.bin, r0.count);
      flush(st.hist[1], r1.bin, r1.count);
      flush(st.hist[2], r2.bin, r2.count);
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (wave == j && active[j]) {
          const uint32_t bin = choose_bin(st, st.hist[cut_group(pre, rk, j)], j, lane);
          if (lane == 0) st.prefix[j] = (pre[j] << (pos - next)) | bin;
        }
      __syncthreads();
      pos = next;
      read_state();
    }
    // collect the keys of each cut's bin and pick the one of its rank
    for (int i = tid; i < m; i += kSelThreads) {
      if (in_bin(hi[i])) {
        const uint64_t key = rank_key(score[n_sink + i], n_sink + i);
#pragma unroll
        for (int j = 0; j < 3; ++j)
          if (lead[j] && (key >> pos) == pre[j])
            reinterpret_cast<uint64_t*>(st.hist[j])[atomicAdd(&st.listed[j], 1u)] = key;
      }
    }
    __syncthreads();
    const int j = wave >> 2;  // four waves per cut
    if (j < 3 && active[j == 0 ? 0 : j == 1 ? 1 : 2]) {
      const int g = j == 0 ? 0 : cut_group(pre, rk, j == 1 ? 1 : 2);
      const uint64_t* list = reinterpret_cast<const uint64_t*>(st.hist[g]);
      const int count = static_cast<int>(st.listed[g]);
      const int i = tid & (kList - 1);
      if (i < count) {
        const uint64_t key = list[i];
        uint32_t above = 0;
        for (int x = 0; x < count; ++x) above += list[x] > key ? 1u : 0u;
        if (above + 1 == st.rank[j]) st.cut[j] = key;
      }
    }
    __syncthreads();
  }

  // classification, four tokens per store: c >= T iff the high word is above
  // T's, or equal with the low word at least T's (read only then)
  uint32_t H[3], L[3];
  bool has[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const uint64_t T = st.cut[j];  // 0 (every key) for a cut of rank m
    H[j] = static_cast<uint32_t>(T >> 32);
    L[j] = static_cast<uint32_t>(T);
    has[j] = cut_rank[j] != 0;
  }
  auto tier_of = [&](int t) -> uint32_t {
    if (t < n_sink) return kFP16;
    const uint32_t w = hi[t - n_sink];
    uint32_t lo = 0;
    if ((has[0] && w == H[0]) || (has[1] && w == H[1]) || (has[2] && w == H[2]))
      lo = static_cast<uint32_t>(rank_key(score[t], t));
    bool ge[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) ge[j] = has[j] && (w > H[j] || (w == H[j] && lo >= L[j]));
    return ge[0] ? kFP16 : ge[1] ? kINT8 : ge[2] ? kINT4 : kDROP;
  };
  typedef uint32_t __attribute__((aligned(1))) u32_any;
  for (int t = 4 * tid; t + 4 <= n; t += 4 * kSelThreads)
    *reinterpret_cast<u32_any*>(tier + t) =
        tier_of(t) | tier_of(t + 1) << 8 | tier_of(t + 2) << 16 | tier_of(t + 3) << 24;
  for (int t = (n & ~3) + tid; t < n; t += kSelThreads) tier[t] = static_cast<uint8_t>(tier_of(t));
}

// The assignment of one score row of any length by one 1024-thread workgroup.
__device__ __forceinline__ void assign_general(const double* __restrict__ score, uint8_t* __restrict__ tier, int n,
                                               int n_sink, int n16, int n8, int n4) {
  __shared__ __attribute__((aligned(16))) SelectState st;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const uint32_t cut_rank[3] = {static_cast<uint32_t>(n16), static_cast<uint32_t>(n16 + n8),
                                static_cast<uint32_t>(n16 + n8 + n4)};
  if (tid < 3) {
    st.prefix[tid] = 0;
    st.rank[tid] = tid == 0 ? cut_rank[0] : tid == 1 ? cut_rank[1] : cut_rank[2];
  }
  __syncthreads();

  int hi_bit = 64;  // digit `pass` is key bits [low, hi_bit)
  for (int pass = 0; pass < kPasses; ++pass) {
    const int low = digit_low_bit(pass);
    const uint32_t mask = (1u << (hi_bit - low)) - 1u;
    if (tid < 3) {
      int grp = tid;
      for (int j = 0; j < tid; ++j)
        if (st.rank[j] != 0 && st.prefix[j] == st.prefix[tid]) { grp = j; break; }
      st.group[tid] = grp;
    }
    for (int i = tid; i < 3 * kBins; i += kSelThreads) (&st.hist[0][0])[i] = 0;
    __syncthreads();
    const bool act0 = st.rank[0] != 0 && st.group[0] == 0;
    const bool act1 = st.rank[1] != 0 && st.group[1] == 1;
    const bool act2 = st.rank[2] != 0 && st.group[2] == 2;
    const uint64_t pre0 = st.prefix[0], pre1 = st.prefix[1], pre2 = st.prefix[2];
    RunCounter r0, r1, r2;
    const uint64_t decided = pass == 0 ? 0ull : (~0ull << hi_bit);
    for (int base = n_sink + tid; base < n; base += kBatch * kSelThreads) {
      double sc[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int t = base + u * kSelThreads;
        sc[u] = t < n ? score[t] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int t = base + u * kSelThreads;
        if (t >= n) break;
        const uint64_t c = rank_key(sc[u], t);
        const uint32_t bin = static_cast<uint32_t>(c >> low) & mask;
        const uint64_t d = c & decided;
        if (act0 && d == pre0) r0.add(st.hist[0], bin);
        if (act1 && d == pre1) r1.add(st.hist[1], bin);
        if (act2 && d == pre2) r2.add(st.hist[2], bin);
      }
    }
    flush(st.hist[0], r0.bin, r0.count);
    flush(st.hist[1], r1.bin, r1.count);
    flush(st.hist[2], r2.bin, r2.count);
    __syncthreads();
    choose_digits(st, low, lane, wave);
    __syncthreads();
    hi_bit = low;
    if ((st.rank[0] | st.rank[1] | st.rank[2]) == 0u) break;  // uniform: every cut is final
  }

  // c >= st.prefix[j] is now cut j (the last digit's bins hold one key each);
  // a cut of rank 0 from the start admits no key.
  const uint64_t T1 = st.prefix[0], T2 = st.prefix[1], T3 = st.prefix[2];
  const bool has1 = cut_rank[0] != 0, has2 = cut_rank[1] != 0, has3 = cut_rank[2] != 0;
  for (int t = tid; t < n; t += kSelThreads) {
    uint8_t tr = kFP16;  // sinks
    if (t >= n_sink) {
      const uint64_t c = rank_key(score[t], t);
      tr = (has1 && c >= T1) ? kFP16 : (has2 && c >= T2) ? kINT8 : (has3 && c >= T3) ? kINT4 : kDROP;
    }
    tier[t] = tr;
  }
}

bool fits_resident(int n, int n_sink) { return n - n_sink <= kResident * kSelThreads; }

// Split form, for rows past the resident form when the caller gives scratch:
// the same digits and digit choices, but each pass is one launch over the
// whole GPU.  sel_pass gives every workgroup kBatch * 1024 consecutive
// non-sink tokens of one row, counts their digits into shared-memory
// histograms and adds the nonzero bins into the row's histogram in device
// memory (integer atomics, so the totals do not depend on the order); the
// workgroup that adds last picks each cut's digit from the totals exactly as
// the one-workgroup form does and clears the histogram of the next pass.  Once
// every cut is final, the remaining passes return at once.  sel_classify then
// assigns every token against the three cuts, so the tier maps equal the
// one-workgroup form's.  Bound by latency: a launch is one round of loads, two
// of atomics, one of the totals and a bin choice.  262144 decayed scores, calls
// back to back: 59 us with a launch for the counts and one for the choice of each
// pass, all six passes, 28 us so; tied scores, which need all six, 60 and 55 us (62
// while the last workgroup read its totals one load after another).  With
// device-wide fences around the ticket, which write back and invalidate the L2, a
// handoff of 4 x 4 x 64 x 262144 gained nothing.
// The rows are those of a grouped map (one length; counts from the group
// table, 8 words per row: sinks, fp16, int8, int4, ...), a single request, or
// the requests of a batched launch.
struct SelScratch {
  uint32_t hist[2][3][kBins];  // per pass parity: the cut groups' digit counts
  uint64_t prefix[3];          // decided key bits of each cut
  uint32_t rank[3];            // remaining rank inside the prefix; 0: the cut is final
  uint32_t ticket;             // workgroups that have added their counts, over all passes
};

// Rows of one shared length n: row r's scores and tiers sit at r * n, its
// counts come from the group table or, for a single row, the arguments.
struct SelRows {
  const double* score;
  uint8_t* tier;
  int n;
  const uint32_t* table;  // per-row counts, or null: the counts below
  int n_sink, n16, n8, n4;
  __device__ __forceinline__ const double* row_score(int row) const { return score + static_cast<size_t>(row) * n; }
  __device__ __forceinline__ uint8_t* row_tier(int row) const { return tier + static_cast<size_t>(row) * n; }
  __device__ __forceinline__ int row_n(int) const { return n; }
  __device__ __forceinline__ void counts(int row, int& s, int& c16, int& c8, int& c4) const {
    if (table != nullptr) {
      const uint32_t* e = table + 8 * row;
      s = static_cast<int>(e[0]);
      c16 = static_cast<int>(e[1]);
      c8 = static_cast<int>(e[2]);
      c4 = static_cast<int>(e[3]);
    } else {
      s = n_sink;
      c16 = n16;
      c8 = n8;
      c4 = n4;
    }
  }
};

// The requests of one batched launch, each with its own length, buffers and
// counts.
struct BatchRows {
  ScoreBatchArgs a;
  __device__ __forceinline__ const double* row_score(int row) const { return a.r[row].score; }
  __device__ __forceinline__ uint8_t* row_tier(int row) const { return a.r[row].tier; }
  __device__ __forceinline__ int row_n(int row) const { return a.r[row].n; }
  __device__ __forceinline__ void counts(int row, int& s, int& c16, int& c8, int& c4) const {
    const ScoreDesc& q = a.r[row];
    s = q.n_sink;
    c16 = q.n16;
    c8 = q.n8;
    c4 = q.n4;
  }
};
static_assert(sizeof(BatchRows) + sizeof(void*) + sizeof(int) <= 4000, "kernel arguments");

// grid: one workgroup (256 threads) per row; the cuts start undecided at
// their ranks
template <typename Rows>
__global__ __launch_bounds__(256) void sel_init(const Rows a, SelScratch* __restrict__ scratch) {
  SelScratch* sc = scratch + blockIdx.x;
  int s, c16, c8, c4;
  a.counts(blockIdx.x, s, c16, c8, c4);
  if (threadIdx.x < 3) {
    sc->prefix[threadIdx.x] = 0;
    sc->rank[threadIdx.x] = static_cast<uint32_t>(threadIdx.x == 0 ? c16 : threadIdx.x == 1 ? c16 + c8 : c16 + c8 + c4);
  }
  if (threadIdx.x == 3) sc->ticket = 0;
  for (int i = threadIdx.x; i < 3 * kBins; i += 256) (&sc->hist[0][0][0])[i] = 0;
}

// grid: (ceil(longest row / (kBatch * 1024)), rows); pass `pass`.
// Workgroups past a row's last non-sink token, and all of a row whose cuts are
// final (the ranks change only after a pass's last ticket is drawn), return.
template <typename Rows>
__global__ __launch_bounds__(kSelThreads) void sel_pass(const Rows a, SelScratch* __restrict__ scratch, int pass) {
  __shared__ __attribute__((aligned(16))) SelectState st;
  __shared__ bool s_last;
  const int row = blockIdx.y;
  SelScratch* sc = scratch + row;
  int n_sink, c16, c8, c4;
  a.counts(row, n_sink, c16, c8, c4);
  const int n = a.row_n(row);
  if (n_sink + static_cast<int>(blockIdx.x) * kBatch * kSelThreads >= n) return;  // uniform per workgroup
  const double* __restrict__ score = a.row_score(row);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint64_t pre[3];
  uint32_t rk[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    pre[j] = sc->prefix[j];
    rk[j] = sc->rank[j];
  }
  if ((rk[0] | rk[1] | rk[2]) == 0u) return;  // uniform per row
  const bool act0 = rk[0] != 0, act1 = rk[1] != 0 && cut_group(pre, rk, 1) == 1,
             act2 = rk[2] != 0 && cut_group(pre, rk, 2) == 2;
  const int low = digit_low_bit(pass), hi_bit = pass == 0 ? 64 : digit_low_bit(pass - 1);
  const uint32_t mask = (1u << (hi_bit - low)) - 1u;
  const uint64_t decided = pass == 0 ? 0ull : (~0ull << hi_bit);
  // this workgroup's tokens: base + u * 1024, u < kBatch
  const int base = n_sink + blockIdx.x * kBatch * kSelThreads + tid;
  double v[kBatch];
#pragma unroll
  for (int u = 0; u < kBatch; ++u) {
    const int t = base + u * kSelThreads;
    v[u] = t < n ? score[t] : 0.0;
  }
  for (int i = tid; i < 3 * kBins; i += kSelThreads) (&st.hist[0][0])[i] = 0;
  __syncthreads();
  if (pass == 0) {
    // every prefix is empty: the first cut of nonzero rank leads the only
    // group, and neighbouring tokens mostly share the exponent digit
    const int lead = act0 ? 0 : act1 ? 1 : 2;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int t = base + u * kSelThreads;
      const uint32_t bin = static_cast<uint32_t>(rank_key(v[u], t) >> low) & mask;
      wave_count(st.hist[lead], t < n, bin, lane);
    }
  } else {
    RunCounter r0, r1, r2;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int t = base + u * kSelThreads;
      if (t >= n) break;
      const uint64_t c = rank_key(v[u], t);
      const uint32_t bin = static_cast<uint32_t>(c >> low) & mask;
      const uint64_t d = c & decided;
      if (act0 && d == pre[0]) r0.add(st.hist[0], bin);
      if (act1 && d == pre[1]) r1.add(st.hist[1], bin);
      if (act2 && d == pre[2]) r2.add(st.hist[2], bin);
    }
    flush(st.hist[0], r0.bin, r0.count);
    flush(st.hist[1], r1.bin, r1.count);
    flush(st.hist[2], r2.bin, r2.count);
  }
  __syncthreads();
  uint32_t* totals = &sc->hist[pass & 1][0][0];
  for (int i = tid; i < 3 * kBins; i += kSelThreads) {
    const uint32_t c = (&st.hist[0][0])[i];
    if (c) atomicAdd(&totals[i], c);
  }

  // the row's last workgroup of this pass chooses the digits: a workgroup draws
  // its ticket when its additions, which are made in device memory, are done
  // (every wave waits for its own), and the last one reads the totals there, by
  // device-scope loads.  No cache holds any of it, so no fence writes back or
  // invalidates an L2.
  // This orders atomics only: a plain store ahead of the ticket would need a
  // release and an acquire.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    const uint32_t per_pass = static_cast<uint32_t>((n - n_sink + kBatch * kSelThreads - 1) / (kBatch * kSelThreads));
    s_last = atomicAdd(&sc->ticket, 1u) + 1u == static_cast<uint32_t>(pass + 1) * per_pass;
  }
  __syncthreads();
  if (!s_last) return;
  constexpr int kPerThread = 3 * kBins / kSelThreads;
  uint32_t sum[kPerThread];  // loaded together: one round trip
#pragma unroll
  for (int u = 0; u < kPerThread; ++u)
    sum[u] = __hip_atomic_load(&totals[tid + u * kSelThreads], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int u = 0; u < kPerThread; ++u) (&st.hist[0][0])[tid + u * kSelThreads] = sum[u];
  if (tid < 3) {
    st.prefix[tid] = tid == 0 ? pre[0] : tid == 1 ? pre[1] : pre[2];
    st.rank[tid] = tid == 0 ? rk[0] : tid == 1 ? rk[1] : rk[2];
    st.group[tid] = cut_group(pre, rk, tid);
  }
  __syncthreads();
  choose_digits(st, low, lane, wave);
  __syncthreads();
  if (tid < 3) {
    sc->prefix[tid] = st.prefix[tid];
    sc->rank[tid] = st.rank[tid];
  }
  // the next pass counts into the other histogram
  uint32_t* next = &sc->hist[(pass + 1) & 1][0][0];
  for (int i = tid; i < 3 * kBins; i += kSelThreads) next[i] = 0;
}

// grid: (ceil(longest row / 1024), rows); c >= sc->prefix[j] is now cut j, and
// a cut of rank 0 from the start admits no key
template <typename Rows>
__global__ __launch_bounds__(kSelThreads) void sel_classify(const Rows a, const SelScratch* __restrict__ scratch) {
  const int row = blockIdx.y, n = a.row_n(row);
  const int t = blockIdx.x * kSelThreads + threadIdx.x;
  if (t >= n) return;
  const SelScratch* sc = scratch + row;
  int n_sink, c16, c8, c4;
  a.counts(row, n_sink, c16, c8, c4);
  const bool has1 = c16 != 0, has2 = c16 + c8 != 0, has3 = c16 + c8 + c4 != 0;
  uint8_t tr = kFP16;  // sinks
  if (t >= n_sink) {
    const uint64_t c = rank_key(a.row_score(row)[t], t);
    tr = (has1 && c >= sc->prefix[0]) ? kFP16 : (has2 && c >= sc->prefix[1]) ? kINT8
         : (has3 && c >= sc->prefix[2])                                       ? kINT4
                                                                               : kDROP;
  }
  a.row_tier(row)[t] = tr;
}

// max_n: the longest row
template <typename Rows>
hipError_t launch_assign_split(const Rows& a, int rows, int max_n, SelScratch* sc, hipStream_t stream) {
  sel_init<<<rows, 256, 0, stream>>>(a, sc);
  hipError_t e = hipGetLastError();
  const int per = kBatch * kSelThreads;
  const dim3 pass_grid((max_n + per - 1) / per, rows);
  for (int pass = 0; pass < kPasses && e == hipSuccess; ++pass) {
    sel_pass<<<pass_grid, kSelThreads, 0, stream>>>(a, sc, pass);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  sel_classify<<<dim3((max_n + kSelThreads - 1) / kSelThreads, rows), kSelThreads, 0, stream>>>(a, sc);
  return hipGetLastError();
}

// Waves per SIMD of a resident launch: two workgroups per CU for the small instance.
template <int RES>
constexpr int resident_waves() { return RES <= kResidentSmall ? 8 : 4; }

template <int RES>
__global__ __launch_bounds__(kSelThreads, resident_waves<RES>()) void assign_tiers(const double* __restrict__ score,
                                                                                  uint8_t* __restrict__ tier, int n,
                                                                                  int n_sink, int n16, int n8,
                                                                                  int n4) {
  assign_resident<RES>(score, tier, n, n_sink, n16, n8, n4);
}

__global__ __launch_bounds__(kSelThreads) void assign_tiers_long(const double* __restrict__ score,
                                                                 uint8_t* __restrict__ tier, int n, int n_sink,
                                                                 int n16, int n8, int n4) {
  assign_general(score, tier, n, n_sink, n16, n8, n4);
}

// grid: one workgroup per group; plan counts from the group table
// (u32 [sinks, fp16, int8, int4, ...], 32 bytes per group).  Rows of at most
// RES * kSelThreads tokens (longer rows take the split form).
template <int RES>
__global__ __launch_bounds__(kSelThreads, resident_waves<RES>()) void assign_tiers_groups(
    const double* __restrict__ score, uint8_t* __restrict__ tier, int n, const uint32_t* __restrict__ group_table) {
  const uint32_t* e = group_table + 8 * blockIdx.x;
  const size_t row = static_cast<size_t>(blockIdx.x) * n;
  assign_resident<RES>(score + row, tier + row, n, static_cast<int>(e[0]), static_cast<int>(e[1]),
                       static_cast<int>(e[2]), static_cast<int>(e[3]));
}

// grid: one workgroup per request of the launch
template <int RES>
__global__ __launch_bounds__(kSelThreads, resident_waves<RES>()) void assign_tiers_batch(const ScoreBatchArgs a) {
  const ScoreDesc& q = a.r[blockIdx.x];
  assign_resident<RES>(q.score, q.tier, q.n, q.n_sink, q.n16, q.n8, q.n4);
}

__global__ __launch_bounds__(kSelThreads) void assign_tiers_batch_long(const ScoreBatchArgs a) {
  const ScoreDesc& q = a.r[blockIdx.x];
  assign_general(q.score, q.tier, q.n, q.n_sink, q.n16, q.n8, q.n4);
}

}  // namespace

bool assign_fits_resident(int32_t n, int32_t n_sink) { return fits_resident(n, n_sink); }

hipError_t launch_assign_batch(const ScoreBatchArgs& a, bool resident, void* scratch, hipStream_t stream) {
  if (!resident && scratch != nullptr) {
    int max_n = 0;
    for (int i = 0; i < a.count; ++i) max_n = a.r[i].n > max_n ? a.r[i].n : max_n;
    return launch_assign_split(BatchRows{a}, a.count, max_n, static_cast<SelScratch*>(scratch), stream);
  }
  int longest = 0;
  for (int i = 0; i < a.count; ++i) longest = max(longest, a.r[i].n - a.r[i].n_sink);
  if (!resident)
    assign_tiers_batch_long<<<a.count, kSelThreads, 0, stream>>>(a);
  else if (longest <= kResidentSmall * kSelThreads)
    assign_tiers_batch<kResidentSmall><<<a.count, kSelThreads, 0, stream>>>(a);
  else
    assign_tiers_batch<kResident><<<a.count, kSelThreads, 0, stream>>>(a);
  return hipGetLastError();
}

uint64_t assign_scratch_bytes(int32_t n, int32_t rows) {
  return fits_resident(n, 0) ? 0 : (static_cast<uint64_t>(rows) * sizeof(SelScratch) + 255) / 256 * 256;
}

hipError_t launch_assign(const Geometry& g, const double* score, uint8_t* tier, void* scratch,
                         hipStream_t stream) {
  if (g.n - g.n_sink <= kResidentSmall * kSelThreads)
    assign_tiers<kResidentSmall><<<1, kSelThreads, 0, stream>>>(score, tier, g.n, g.n_sink, g.n16, g.n8, g.n4);
  else if (fits_resident(g.n, g.n_sink))
    assign_tiers<kResident><<<1, kSelThreads, 0, stream>>>(score, tier, g.n, g.n_sink, g.n16, g.n8, g.n4);
  else if (scratch != nullptr)
    return launch_assign_split(SelRows{score, tier, g.n, nullptr, g.n_sink, g.n16, g.n8, g.n4}, 1, g.n,
                               static_cast<SelScratch*>(scratch), stream);
  else
    assign_tiers_long<<<1, kSelThreads, 0, stream>>>(score, tier, g.n, g.n_sink, g.n16, g.n8, g.n4);
  return hipGetLastError();
}

hipError_t launch_assign_groups(int32_t G, int32_t n, const uint32_t* group_table, const double* score,
                                uint8_t* tier, void* scratch, hipStream_t stream) {
  if (!fits_resident(n, 0)) {
    if (scratch == nullptr) return hipErrorInvalidValue;
    return launch_assign_split(SelRows{score, tier, n, group_table, 0, 0, 0, 0}, G, n,
                               static_cast<SelScratch*>(scratch), stream);
  }
  if (n <= kResidentSmall * kSelThreads)
    assign_tiers_groups<kResidentSmall><<<G, kSelThreads, 0, stream>>>(score, tier, n, group_table);
  else
    assign_tiers_groups<kResident><<<G, kSelThreads, 0, stream>>>(score, tier, n, group_table);
  return hipGetLastError();
}

}  // namespace skv
