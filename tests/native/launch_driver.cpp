// Records the launches that the library's row calls make (no device: the HIP
// launch entry points are replaced here) and checks them against the limits of
// a grid: fewer than 2^32 threads along x.  The largest admitted requests of
// many (layer, head) pairs need several launches of one row kernel; their
// pieces must follow one another without a gap or an overlap.  Requests of at
// most 32 tokens get one workgroup per chunk, as a second would have no token.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include <hip/hip_runtime.h>

#include "skv.h"

namespace {

struct Launch {
  const void* kernel;
  uint64_t blocks, threads, first;
};
std::vector<Launch> launches;
size_t lead = 0;  // launches of the present call before its row kernels (init, prep, check)
hipError_t last = hipSuccess;

void begin(size_t before_rows) {
  launches.clear();
  lead = before_rows;
}

int fail(const char* what, int d, int n, int variant) {
  printf("%s: d=%d n=%d variant=%d\n", what, d, n, variant);
  return 1;
}

// Argument 1 of a row kernel is its first flat workgroup.  A kernel covers all
// chunks or, with per-channel keys, those of K (one workgroup each) or of V; a
// chunk is one, two, four or eight workgroups.
int check(uint64_t chunks, int d, int n, int variant) {
  if (launches.size() <= lead) return fail("no row launch", d, n, variant);
  const uint64_t per_kernel = variant & SKV_QUANT_CHANNEL && launches[lead].kernel != launches.back().kernel ? chunks / 2 : chunks;
  uint64_t done = 0;
  for (size_t i = lead; i < launches.size(); ++i) {
    const Launch& l = launches[i];
    if (l.first != done) return fail("a piece does not follow the one before", d, n, variant);
    if (l.blocks * l.threads >= 1ull << 32) return fail("a grid past the limit", d, n, variant);
    done += l.blocks;
    if (i + 1 == launches.size() || launches[i + 1].kernel != l.kernel) {
      const uint64_t split = done / per_kernel;
      if (done % per_kernel != 0 || split < 1 || split > 8 || (split & (split - 1)) != 0)
        return fail("the chunks are not covered", d, n, variant);
      if (n <= 32 && split != 1) return fail("workgroups without a token", d, n, variant);  // a part has at least 32
      done = 0;
    }
  }
  return 0;
}

}  // namespace

extern "C" hipError_t hipLaunchKernel(const void* kernel, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  const bool fits = static_cast<uint64_t>(grid.x) * block.x < 1ull << 32;
  last = fits ? hipSuccess : hipErrorInvalidConfiguration;
  launches.push_back(Launch{kernel, grid.x, block.x, launches.size() < lead ? 0 : *static_cast<uint32_t*>(args[1])});
  return last;
}
// what <<<...>>> expands to, without a device
static dim3 cfg_grid, cfg_block;
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  cfg_grid = grid;
  cfg_block = block;
  return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = cfg_grid;
  *block = cfg_block;
  *shared = 0;
  *stream = nullptr;
  return hipSuccess;
}
extern "C" hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}

int main() {
  uint8_t* const p = reinterpret_cast<uint8_t*>(uintptr_t{1} << 40);  // aligned; never read on the host
  const uint64_t all = ~0ull;
  int calls = 0;
  for (int d : {32, 64, 128, 256}) {
    const int most = 65536 / (d / 32);  // 8 MiB of K and V per pair: more than any device holds
    for (int n : {1, 32, 257, most / 4 + 1, most / 2 - 255, most / 2, most}) {
      for (int variant : {0, SKV_QUANT_ASYM | SKV_QUANT_FP16, SKV_QUANT_CHANNEL | SKV_QUANT_ASYM}) {
        skv_config c = {};
        c.num_layers = 64;  // the most pairs a configuration may have
        c.num_kv_heads = 1024;
        c.head_dim = d;
        c.num_tokens = n;
        c.budget = n == 1 ? 1.0f : 0.3f;
        c.num_sink = 0;
        c.num_tiers = 3;
        c.score_mode = SKV_SCORE_KVNORM;
        c.quant_int8 = c.quant_int4 = variant;
        const uint64_t per_pair = 2ull * static_cast<uint64_t>((n + 255) / 256);
        uint64_t chunks = 65536 * per_pair;
        begin(1);
        if (skv_pack(&c, p, p, p, p, all, nullptr, nullptr) != SKV_OK) return fail("skv_pack refused", d, n, variant);
        if (check(chunks, d, n, variant)) return 1;
        begin(1);
        if (skv_unpack(&c, p, all, p, p, reinterpret_cast<int32_t*>(p), n, 16, reinterpret_cast<uint32_t*>(p),
                       nullptr) != SKV_OK)
          return fail("skv_unpack refused", d, n, variant);
        if (check(chunks, d, n, variant)) return 1;
        calls += 2;
        if (variant != 0) continue;
        c.num_layers = 65535;  // the most pairs a grouped call takes
        c.num_kv_heads = 1;
        chunks = 65535 * per_pair;
        const skv_group_spec g = {SKV_GROUP_LAYER, 0, nullptr};
        begin(2);
        if (skv_pack_groups(&c, &g, p, p, p, p, p, all, nullptr, nullptr) != SKV_OK)
          return fail("skv_pack_groups refused", d, n, variant);
        if (check(chunks, d, n, variant)) return 1;
        begin(2);
        if (skv_unpack_groups(&c, &g, p, p, all, p, p, reinterpret_cast<int32_t*>(p), n, 16,
                              reinterpret_cast<uint32_t*>(p), nullptr) != SKV_OK)
          return fail("skv_unpack_groups refused", d, n, variant);
        if (check(chunks, d, n, variant)) return 1;
        calls += 2;
      }
    }
  }
  printf("ok %d calls\n", calls);
  return 0;
}
