// Host-side check of the attention launchers (attn_bf16.hip, attn_f32.hip), built by
// the CPU test suite from their host code and the stand-ins below for the HIP runtime:
// a launch that fails ends the call with its error and nothing is launched after it
// (the kernels after a pre-pass read what it wrote), and every launch stays below
// 2^32 threads, also on the plans with the most rows.  Exit status 0 means pass.
#include <cstdio>
#include <string>
#include <vector>

#include "tra_internal.h"

namespace {
int n_launched = 0, fail_at = -1;
bool too_many_threads = false;
hipError_t last = hipSuccess;
dim3 cfg_grid, cfg_block;
size_t cfg_lds = 0;
hipStream_t cfg_stream = nullptr;
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h = nullptr; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *s = cfg_stream;
  return hipSuccess;
}
// (a later launch that succeeds hides an earlier one's error from hipGetLastError)
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  if ((unsigned long long)grid.x * grid.y * grid.z * block.x >= 1ull << 32) too_many_threads = true;
  last = n_launched++ == fail_at ? hipErrorInvalidConfiguration : hipSuccess;
  return last;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 2;
  return hipSuccess;
}
}

namespace {

int failures = 0;

void expect(bool ok, const std::string& what) {
  if (ok) return;
  std::printf("FAIL %s\n", what.c_str());
  ++failures;
}

tra_plan_s make_plan(int dtype, int batch, int heads, int NB, int d, int dist, int text) {
  tra_plan_s p;
  p.cfg = tra_config{};
  p.cfg.batch = batch; p.cfg.heads = heads; p.cfg.head_dim = d; p.cfg.block = 128; p.cfg.dtype = dtype;
  p.cfg.frames = 4; p.cfg.height = 30; p.cfg.width = 52; p.cfg.distance = dist; p.cfg.text_tokens = text;
  p.S = NB * 128 - 5;
  p.N = p.S - text;
  p.NB = p.NBa = NB;
  p.rows = p.rowsa = batch * heads * NB;
  p.n_pad = p.n_pada = NB * 128;
  p.n_cap = 100;
  p.n_cu = 256;
  p.split_wg_cap = tra::k64_sparse_grid_cap(p);
  tra::split_capacities(p.split_wg_cap, p.rows, NB, d, &p.units_cap, &p.splits_cap, &p.slots_cap);
  tra::dense_capacities(p, &p.dense_splits, &p.dense_slots);
  return p;
}

int x[4];  // something to point at: nothing on the host reads it
hipError_t call(const tra_plan_s& p, const tra::AttnArgs& a) {
  n_launched = 0;
  last = hipSuccess;
  return p.cfg.dtype == TRA_BF16 ? tra::launch_attention_bf16(p, a, nullptr) : tra::launch_attention_f32(p, a, nullptr);
}

tra::AttnArgs args(const char* kind, bool lse) {
  const std::string k = kind;
  tra::AttnArgs a{};
  a.q = a.k = x;
  float* f = (float*)x;
  if (k != "entropy") { a.v = x; a.o = x; }
  if (k == "entropy" || k == "fused") a.entropy = f;
  if (lse && k != "entropy" && k != "fused") a.lse = f;
  if (k == "sparse" || k == "token") { a.sparse = true; a.cnt = a.cols = x; }
  if (k == "token") a.radius_sq = x;
  return a;
}

}  // namespace

int main() {
  const char* kinds[] = {"dense", "entropy", "fused", "sparse", "token"};
  int most = 0;
  for (int dtype : {TRA_BF16, TRA_FP32})
    for (int d : {64, 128})
      for (int dist : {TRA_DIST_2D, TRA_DIST_1D})
        for (int text : {0, 3})
          for (const char* kind : kinds)
            // few rows; short rows, never cut; rows of which some are cut (dense: all but five)
            for (const auto& s : std::vector<std::pair<int, int>>{{2, 8}, {40, 16}, {7, 159}})
              for (bool lse : {false, true}) {
                const tra_plan_s p = make_plan(dtype, 1, s.first, s.second, d, dist, text);
                const tra::AttnArgs a = args(kind, lse);
                const std::string what = std::string(kind) + " dtype " + std::to_string(dtype) + " d " + std::to_string(d) +
                                         " heads " + std::to_string(s.first) + " blocks " + std::to_string(s.second);
                fail_at = -1;
                expect(call(p, a) == hipSuccess, what);
                const int n = n_launched;
                most = std::max(most, n);
                expect(n > 0, what + ": no launch");
                for (fail_at = 0; fail_at < n; ++fail_at) {
                  const int k = fail_at;
                  expect(call(p, a) == hipErrorInvalidConfiguration, what + ": error of launch " + std::to_string(k) + " lost");
                  expect(n_launched == k + 1, what + ": launches after a failed one");
                }
                fail_at = -1;
              }
  expect(most == 3, "calls of three launches (pre-pass, attention, merge)");
  // 2^23 one-block heads, just below the plans' limit of 2^31 padded tokens
  for (int dtype : {TRA_BF16, TRA_FP32})
    for (const char* kind : kinds) {
      const tra_plan_s p = make_plan(dtype, 1 << 12, (1 << 12) - 1, 1, 64, TRA_DIST_2D, 0);
      too_many_threads = false;
      expect(call(p, args(kind, true)) == hipSuccess, kind);
      expect(!too_many_threads, std::string(kind) + " dtype " + std::to_string(dtype) + ": 2^32 threads in a launch");
    }
  if (failures) return 1;
  std::printf("launches: ok\n");
  return 0;
}
