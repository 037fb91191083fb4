// The library's host side (api.cpp, devmem.cpp, analysis.cpp, strips.cpp) on the
// CPU: a stand-in for the HIP runtime whose device memory is the host's, with
// failures to order, and stand-ins for the launchers that note their names.
// Results are not computed; what is checked is which form a call takes, what it
// leaves allocated and what error it leaves behind.
#include <hip/hip_runtime_api.h>

#include <chrono>
#include <cstdlib>
#include <cstring>
#include <future>
#include <map>
#include <set>
#include <string>

#include "analysis.hpp"
#include "analysis_gpu.hpp"
#include "column.hpp"
#include "devmem.hpp"
#include "kernels.hpp"
#include "probe.hpp"
#include "strips.hpp"

using namespace sptrsv;

namespace {

std::map<void*, size_t> g_live;
hipError_t g_last = hipSuccess;
int64_t g_fail_from = INT64_MAX;   // allocations of at least this many bytes fail
int g_fail_next = 0;               // and so do the next so many of any size
bool g_capturing = false;
std::string g_log;
int64_t g_npub = 0;                // published values of every strip copy, 0: as many as rows
int64_t g_strip_bytes = 1 << 16;   // size of every strip copy
int g_strip_error = 0;             // what the construction of one reports
void* g_xp = nullptr;              // the solution buffer filled last
int g_probe_free = 0;              // the next free tries an allocation of another thread:
                                   // 2 it went through meanwhile, 3 it had to wait
std::future<void> g_other;
int g_handles = 0;                 // events, streams and graphs are numbers

hipError_t fail(hipError_t e) { return g_last = e; }
hipError_t note(const char* what) {
  if (!g_log.empty()) g_log += ' ';
  g_log += what;
  return hipGetLastError();        // as a launcher ends
}

}  // namespace

extern "C" {

void model_fail_from(int64_t bytes) { g_fail_from = bytes < 0 ? INT64_MAX : bytes; }
void model_fail_next(int count) { g_fail_next = count; }
void model_capture(int on) { g_capturing = on != 0; }
void model_npub(int64_t npub) { g_npub = npub; }
void model_strip_bytes(int64_t bytes) { g_strip_bytes = bytes; }
void model_strip_error(int status) { g_strip_error = status; }
const char* model_log() {
  static std::string out;
  out.swap(g_log);
  g_log.clear();
  return out.c_str();
}
void* model_xp() { return g_xp; }
int model_last_error() { return static_cast<int>(hipGetLastError()); }
int64_t model_live_bytes() {
  int64_t b = 0;
  for (auto& kv : g_live) b += static_cast<int64_t>(kv.second);
  return b;
}
int model_is_live(void* p) {
  for (auto& kv : g_live)
    if (p >= kv.first && p < static_cast<char*>(kv.first) + kv.second) return 1;
  return 0;
}
void* model_alloc(int64_t bytes) {
  void* p = nullptr;
  return dev_alloc(&p, bytes) == hipSuccess ? p : nullptr;
}
void model_free(void* p) { dev_free(p); }
void model_reset() {                // what a device reset leaves of the allocations
  for (auto& kv : g_live) std::free(kv.first);
  g_live.clear();
}
void model_probe_free() { g_probe_free = 1; }
int model_probed() {
  if (g_other.valid()) g_other.get();
  return g_probe_free;
}

// -------------------------------------------------------------- the runtime
hipError_t hipMalloc(void** p, size_t bytes) {
  if (g_capturing) return fail(hipErrorStreamCaptureUnsupported);
  if (g_fail_next > 0 || static_cast<int64_t>(bytes) >= g_fail_from) {
    if (g_fail_next > 0) --g_fail_next;
    return fail(hipErrorOutOfMemory);
  }
  *p = std::calloc(1, bytes + 64);
  g_live[*p] = bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  if (g_probe_free == 1 && g_live.count(p) && g_live[p] > 1000) {
    g_probe_free = 0;
    g_other = std::async(std::launch::async, [] { dev_free(model_alloc(1 << 20)); });
    g_probe_free = g_other.wait_for(std::chrono::seconds(2)) == std::future_status::ready ? 2 : 3;
  }
  if (g_capturing) return fail(hipErrorStreamCaptureUnsupported);
  auto it = g_live.find(p);
  if (it == g_live.end()) return fail(hipErrorInvalidValue);
  g_live.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  for (auto& kv : g_live)
    if (p >= kv.first && p < static_cast<char*>(kv.first) + kv.second) {
      *base = kv.first;
      *size = kv.second;
      return hipSuccess;
    }
  return fail(hipErrorNotFound);
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  return hipMemcpy(d, s, n, k);
}
hipError_t hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 65536;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(static_cast<intptr_t>(++g_handles));
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  // strips are the fastest schedule here
  *ms = g_log.size() >= 6 && g_log.compare(g_log.size() - 6, 6, "strips") == 0 ? 0.5f : 1.0f;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  g_capturing = true;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  g_capturing = false;
  *g = reinterpret_cast<hipGraph_t>(static_cast<intptr_t>(++g_handles));
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *x = reinterpret_cast<hipGraphExec_t>(static_cast<intptr_t>(++g_handles));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"

// ------------------------------------------------------------ the launchers
namespace sptrsv {

int device_analysis(int, int64_t, const int*, const int*, bool, bool, int,
                    const std::vector<std::vector<StripGrid>>&, int64_t, hipStream_t,
                    DeviceAnalysis&) {
  return kErrNotSupported;
}
void free_device_analysis(DeviceAnalysis&) {}
int device_transpose(int, int64_t, const int*, const int*, hipStream_t, int**, int**, int**) {
  return kErrNotSupported;
}
int device_value_sources(int, int64_t, const int*, const int*, int64_t, const int*,
                         DeviceAnalysis&, hipStream_t) {
  return kErrNotSupported;
}
int device_concat(const std::vector<ConcatSystem>&, int, int*, int*, void*, hipStream_t) {
  return kErrNotSupported;
}
hipError_t launch_pingpong(int*, int*, int, int, int, long long*, int*, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_init_scratch(DevScratch, int, hipStream_t) { return hipGetLastError(); }
hipError_t launch_row_pos(int, const int*, int*, hipStream_t) { return hipGetLastError(); }
hipError_t launch_strip_lanes(const DevChunks&, unsigned char*, hipStream_t) {
  return hipGetLastError();
}

hipError_t launch_strip_offsets(int, int64_t, const int* rp, const int* col, int nsys,
                                const int* row0, int* table, int* full, hipStream_t) {
  (void)note("offsets");
  for (int s = 0; s < nsys; ++s) {
    std::set<int> d;
    for (int i = row0[s]; i < row0[s + 1]; ++i)
      for (int e = rp[i]; e < rp[i + 1]; ++e)
        if (col[e] != i) d.insert(std::abs(col[e] - i));
    int q = 0;
    for (int v : d) {
      if (q == kStripTable) full[s] = 1;
      else table[s * kStripTable + q++] = v;
    }
  }
  return hipGetLastError();
}

int build_strips(const DevPlan& p, const std::vector<StripGrid>& grids, int max_len,
                 const unsigned char* lanes_lg, int vb, hipStream_t, DevStrips& out) {
  out = DevStrips();
  DevStrips t;
  t.acc = lanes_lg ? 4 : 1;
  t.entries = t.acc == 1 ? std::max(2, max_len) : max_len <= 13 ? 13 : 15;
  t.words = (t.entries + 1) * (vb / 4) + (t.entries + 1) / 2;
  for (const StripGrid& g : grids) t.nstrips += g.n > 0 ? g.nbu * g.nbv : 0;
  t.nrec = (p.n + 63) / 64;
  t.npub = g_npub ? g_npub : p.n;
  if (g_strip_error) return g_strip_error;
  if (dev_alloc(&t.mem, g_strip_bytes) != hipSuccess) return kErrOom;
  if (hipGetLastError() != hipSuccess) return kErrHip;
  out = t;
  return kOk;
}
void free_strips(DevStrips& t) {
  dev_free(t.mem);
  t = DevStrips();
}

template <typename T> hipError_t launch_gather(const DevPlan&, const T*, int*, hipStream_t) {
  return note("gather");
}
template <typename T>
hipError_t launch_strip_gather(const DevPlan&, const DevStrips&, hipStream_t) {
  return note("strip_gather");
}
template <typename T> hipError_t launch_push_gather(const DevPlan&, const DevPush&, hipStream_t) {
  return note("push_gather");
}
template <typename T> hipError_t launch_fill_sentinel(T* xp, int64_t count, int*, hipStream_t) {
  if (count > 0) xp[count - 1] = xp[0] = T(0);   // both ends are the buffer's own
  g_xp = xp;
  return note("fill");
}
template <typename T> hipError_t launch_strip_solve(const StripSolveArgs&, hipStream_t) {
  return note("strips");
}
template <typename T>
hipError_t launch_multi_in(int, int, int, const T*, const int*, T*, T*, bool, int*, hipStream_t) {
  return note("multi_in");
}
template <typename T>
hipError_t launch_multi_out(int, int, int, const T*, const int*, T*, hipStream_t) {
  return note("multi_out");
}
template <typename T> hipError_t launch_level(const SolveArgs&, int, int, hipStream_t) {
  return note("level");
}
template <typename T> hipError_t launch_level_flat(const SolveArgs&, int, int, hipStream_t) {
  return note("level");
}
template <typename T> hipError_t launch_self_value(const SolveArgs&, hipStream_t) {
  return note("ticket");
}
template <typename T> hipError_t launch_self_flag(const SolveArgs&, hipStream_t) {
  return note("flag");
}
template <typename T> hipError_t launch_self_static(const SolveArgs& a, hipStream_t) {
  return note(a.nrhs == 1 && a.early ? "static_by_row" : "static");
}
template <typename T>
hipError_t launch_block(const SolveArgs&, const int*, const int*, const int*, int, int, int,
                        hipStream_t) {
  return note("block");
}
template <typename T>
hipError_t launch_block_res(const SolveArgs&, const int*, const int*, int, int, int, hipStream_t) {
  return note("block");
}
template <typename T>
hipError_t launch_grad_vals(int, const int*, const int*, int, const T*, const T*, T*, hipStream_t) {
  return note("grad");
}
template <typename T> hipError_t launch_column_init(const ColumnArgs&, hipStream_t) {
  return hipGetLastError();
}
template <typename T> hipError_t launch_column_level(const ColumnArgs&, int, int, hipStream_t) {
  return note("column_level");
}
template <typename T> hipError_t launch_column_self(const ColumnArgs&, hipStream_t) {
  return note("column_self");
}
template <typename T> int self_value_blocks_per_cu(int) { return 8; }
template <typename T> int self_flag_blocks_per_cu(int) { return 8; }
template <typename T> int self_static_blocks_per_cu(int) { return 8; }
template <typename T> int self_multi_blocks_per_cu(int, int) { return 8; }
template <typename T> int column_self_blocks_per_cu(int) { return 8; }
template <typename T> int strip_blocks_per_cu(const DevStrips&, int) { return 4; }

#define MODEL_INSTANTIATE(T)                                                                       \
  template hipError_t launch_gather<T>(const DevPlan&, const T*, int*, hipStream_t);               \
  template hipError_t launch_strip_gather<T>(const DevPlan&, const DevStrips&, hipStream_t);       \
  template hipError_t launch_push_gather<T>(const DevPlan&, const DevPush&, hipStream_t);          \
  template hipError_t launch_fill_sentinel<T>(T*, int64_t, int*, hipStream_t);                     \
  template hipError_t launch_strip_solve<T>(const StripSolveArgs&, hipStream_t);                   \
  template hipError_t launch_multi_in<T>(int, int, int, const T*, const int*, T*, T*, bool, int*,  \
                                         hipStream_t);                                             \
  template hipError_t launch_multi_out<T>(int, int, int, const T*, const int*, T*, hipStream_t);   \
  template hipError_t launch_level<T>(const SolveArgs&, int, int, hipStream_t);                    \
  template hipError_t launch_level_flat<T>(const SolveArgs&, int, int, hipStream_t);               \
  template hipError_t launch_self_value<T>(const SolveArgs&, hipStream_t);                         \
  template hipError_t launch_self_flag<T>(const SolveArgs&, hipStream_t);                          \
  template hipError_t launch_self_static<T>(const SolveArgs&, hipStream_t);                        \
  template hipError_t launch_block<T>(const SolveArgs&, const int*, const int*, const int*, int,   \
                                      int, int, hipStream_t);                                      \
  template hipError_t launch_block_res<T>(const SolveArgs&, const int*, const int*, int, int, int, \
                                          hipStream_t);                                            \
  template hipError_t launch_grad_vals<T>(int, const int*, const int*, int, const T*, const T*,    \
                                          T*, hipStream_t);                                        \
  template hipError_t launch_column_init<T>(const ColumnArgs&, hipStream_t);                       \
  template hipError_t launch_column_level<T>(const ColumnArgs&, int, int, hipStream_t);            \
  template hipError_t launch_column_self<T>(const ColumnArgs&, hipStream_t);                       \
  template int self_value_blocks_per_cu<T>(int);                                                   \
  template int self_flag_blocks_per_cu<T>(int);                                                    \
  template int self_static_blocks_per_cu<T>(int);                                                  \
  template int self_multi_blocks_per_cu<T>(int, int);                                              \
  template int column_self_blocks_per_cu<T>(int);                                                  \
  template int strip_blocks_per_cu<T>(const DevStrips&, int);

MODEL_INSTANTIATE(double)
MODEL_INSTANTIATE(float)

}  // namespace sptrsv
