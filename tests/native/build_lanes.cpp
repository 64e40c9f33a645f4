// Stream order of prism_build_smatrix with a HIP runtime and kernel launchers
// that only record: every operation queued on any stream has to come before
// whatever the caller queues next on its own stream, also when a launch fails.
// Compiled with plan.cpp by test_build_lanes.py; no GPU and no HIP library.
//
// argv: n, slices, f, bytes of workspace beyond the minimum, failing launch
// (-1: none). Prints "<status> <streams used> <launches> <ordered 0/1> <states
// in bounds and apart 0/1> <planes written once 0/1>".
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>

#include "kernels.hpp"
#include "prism.h"

namespace {

using Clock = std::map<void*, long>;  // per stream: operations known to be complete
std::map<void*, Clock> g_stream;
std::map<void*, Clock> g_event;
long g_launches = 0, g_fail_at = -1;
char g_handles[64];
int g_handle = 0;

// device addresses: never read, only compared
const uintptr_t kWs = uintptr_t(1) << 32, kS = uintptr_t(1) << 44;
std::map<void*, std::pair<uintptr_t, uintptr_t>> g_state;  // per stream: lowest, highest address
std::vector<int> g_planes;                                 // times each beam's plane was written

void state_used(const void* p, size_t bytes, void* st) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = a + bytes;
  auto it = g_state.emplace(st, std::make_pair(a, b)).first;
  if (a < it->second.first) it->second.first = a;
  if (b > it->second.second) it->second.second = b;
}
size_t wave_bytes(int n) { return (size_t)n * (n / 2) * sizeof(float2); }

void op(void* st) { ++g_stream[st][st]; }
hipError_t launch(hipStream_t st) {
  if (g_launches++ == g_fail_at) return hipErrorLaunchFailure;
  op(st);
  return hipSuccess;
}

}  // namespace

extern "C" {
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t st) {
  op(st);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(&g_handles[g_handle++]);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(&g_handles[g_handle++]);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  g_event[e] = g_stream[st];
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
  for (auto& k : g_event[e]) {
    long& mine = g_stream[st][k.first];
    if (k.second > mine) mine = k.second;
  }
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "recorded"; }
}

namespace prism {
hipError_t launch_twiddles(float2*, int, hipStream_t st) { return launch(st); }
hipError_t launch_transmission(const float*, float2*, size_t, float, hipStream_t st) {
  return launch(st);
}
hipError_t launch_prop_lut(float2*, int, int, const double*, double, double, hipStream_t st) {
  return launch(st);
}
hipError_t launch_probe_init(float2*, const double*, int, int, int, const ProbeOptics&,
                             const int2*, const float2*, hipStream_t st) {
  return launch(st);
}
int four_step_radix(int n) { return n == 1024 ? 32 : (n == 256 ? 16 : 0); }
hipError_t launch_twiddles2(float2*, int, hipStream_t st) { return launch(st); }
hipError_t launch_row_pass(float2* state, int nwaves, int n, const float2*, const float2*,
                           const float2*, const LaunchTuning&, hipStream_t st, const BeamWaves*,
                           const float2* const*, size_t, bool) {
  state_used(state, nwaves * wave_bytes(n), st);
  return launch(st);
}
hipError_t launch_col_pass(float2* state, int nwaves, int n, const float2*, const float2*,
                           const float2*, const LaunchTuning&, hipStream_t st, bool) {
  state_used(state, nwaves * wave_bytes(n), st);
  return launch(st);
}
bool few_waves(int, int) { return false; }
hipError_t launch_col_detect(const float2*, int, int, const float2*, const float2*, const DetBins&,
                             double*, hipStream_t st) {
  return launch(st);
}
int col_tiles(int n) { return n / 16; }
hipError_t launch_reduce_partials(const double*, int, int, int, double*, OutAcc, hipStream_t st) {
  return launch(st);
}
hipError_t launch_extract(const float2* state, int nwaves, int n, float2* S, const float2*,
                          hipStream_t st) {
  state_used(state, nwaves * wave_bytes(n), st);
  const size_t first = (reinterpret_cast<uintptr_t>(S) - kS) / (wave_bytes(n) / 2);
  for (int k = 0; k < nwaves; ++k)
    if (first + k < g_planes.size()) ++g_planes[first + k];
  return launch(st);
}
int contract_tile_slots(int, int, int, int, Prec) { return 1; }
int contract_group(int, Prec) { return 16; }
hipError_t launch_s16_scale(const float2*, const ActiveBeam*, int, int, float*, float*,
                            hipStream_t st) {
  return launch(st);
}
hipError_t launch_s16_pack(const float2*, const ActiveBeam*, int, int, int, const float*,
                           const int2*, int, int, void*, Prec, hipStream_t st) {
  return launch(st);
}
hipError_t launch_alpha16(const double*, int, int, const ActiveBeam*, int, int, int, int, int,
                          const ProbeOptics&, const float*, int, void*, int2*, Prec,
                          hipStream_t st) {
  return launch(st);
}
hipError_t launch_contract16(const ContractSegs&, int, int, Prec, int, hipStream_t st) {
  return launch(st);
}
int window_big_tiles(int w) { return w / 16; }
hipError_t launch_window_big(float2*, int, int, const float2*, int, const DetBins&, double*,
                             float*, OutAcc, hipStream_t st) {
  return launch(st);
}
hipError_t launch_window_cbed(const float2*, const WindowSegs&, int, const float2*,
                              hipStream_t st) {
  return launch(st);
}
hipError_t launch_window_detect(const float2*, const WindowSegs&, int, const float2*,
                                hipStream_t st) {
  return launch(st);
}
}  // namespace prism

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const int n = atoi(argv[1]), H = atoi(argv[2]), f = atoi(argv[3]);
  const size_t more = strtoull(argv[4], nullptr, 10);
  std::vector<double> thick(H, 2.0);
  const prism_geometry geo{n, 0.1 * n, 80.0, H, thick.data()};
  prism_plan* plan = nullptr;
  if (prism_plan_create(&plan, &geo)) return 3;
  double amax = 0.0;
  size_t pref = 0, least = 0, sbytes = 0;
  float phase = 0.f;  // device addresses are never read here
  if (prism_alpha_max(plan, f, 20.0, &amax) || prism_smatrix_bytes(plan, f, amax, &sbytes) ||
      prism_build_workspace_bytes(plan, f, amax, &pref, &least) ||
      prism_set_potential_slices(plan, &phase))
    return 4;
  g_fail_at = atol(argv[5]);
  g_planes.assign(sbytes / (wave_bytes(n) / 2), 0);
  char caller;
  hipStream_t st = reinterpret_cast<hipStream_t>(&caller);
  const int status =
      prism_build_smatrix(plan, f, amax, reinterpret_cast<void*>(kS), sbytes,
                          reinterpret_cast<void*>(kWs), least + more, st);
  int used = 0, ordered = 1;
  for (auto& s : g_stream) {
    const long count = s.second[s.first];
    used += count > 0;
    if (g_stream[st][s.first] != count) ordered = 0;
  }
  int apart = 1, once = 1;
  uintptr_t end = kWs;
  std::map<uintptr_t, uintptr_t> ranges;
  for (auto& r : g_state) ranges.insert(r.second);
  for (auto& r : ranges) {
    if (r.first < end) apart = 0;
    end = r.second;
  }
  if (ranges.size() != g_state.size() || end > kWs + least + more) apart = 0;
  for (int k : g_planes) once = once && k == 1;
  printf("%d %d %ld %d %d %d\n", status, used, g_launches, ordered, apart, once);
  prism_plan_destroy(plan);
  return 0;
}
