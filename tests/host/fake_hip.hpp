// A HIP runtime for host tests of the library's plan code: device addresses are handed out but
// have no memory behind them, kernels and copies do nothing, and every call is recorded. The
// definitions below take the place of libamdhip64's in a program that links libfockmi.so.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

namespace fake {

struct Op {
  enum Kind { Launch, Record, Wait, Other } kind;
  hipStream_t stream;
  std::string name;   // kernel
  void* event;
  long thread;
};

struct State {
  std::recursive_mutex mu;
  std::map<uintptr_t, size_t> live;       // device allocations
  std::vector<uintptr_t> freed;
  uintptr_t next = uintptr_t(1) << 40;
  size_t limit = ~size_t(0);              // bytes of device memory
  size_t mallocs = 0, bad_mallocs = 0;    // bad: under capture
  std::set<hipStream_t> capturing;
  std::map<const void*, std::string> kernels;
  std::vector<Op> ops;
  std::map<void*, bool> events;           // live events: recorded or not
  size_t used() const {
    size_t n = 0;
    for (auto& a : live) n += a.second;
    return n;
  }
};
inline State& st() {
  static State* s = new State;  // outlives every static destructor
  return *s;
}

inline hipStream_t stream(int i) { return (hipStream_t)(uintptr_t)(0x1000 * (i + 1)); }
// an array of the caller's, never freed and apart from every other
inline void* user(size_t bytes) {
  State& s = st();
  void* p = (void*)s.next;
  s.next += (bytes + 0xfffff) / 0x100000 * 0x100000;
  return p;
}
inline size_t launches(const std::string& part, size_t from = 0) {
  size_t n = 0;
  for (size_t i = from; i < st().ops.size(); ++i)
    n += st().ops[i].kind == Op::Launch && st().ops[i].name.find(part) != std::string::npos;
  return n;
}
inline void push(Op::Kind k, hipStream_t q, const std::string& name = "", void* ev = nullptr) {
  static long next_thread = 0;
  thread_local long me = ++next_thread;
  std::lock_guard<std::recursive_mutex> l(st().mu);
  st().ops.push_back(Op{k, q, name, ev, me});
}

}  // namespace fake

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  fake::st().kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

static thread_local struct {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} call_cfg;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t q) {
  call_cfg = {g, b, sh, q};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, hipStream_t* q) {
  *g = call_cfg.grid, *b = call_cfg.block, *sh = call_cfg.shared, *q = call_cfg.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t q) {
  fake::push(fake::Op::Launch, q, fake::st().kernels[f]);
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) {
  fake::State& s = fake::st();
  std::lock_guard<std::recursive_mutex> l(s.mu);
  if (!s.capturing.empty()) {
    ++s.bad_mallocs;
    return hipErrorStreamCaptureUnsupported;
  }
  if (n > s.limit || s.used() > s.limit - n) return hipErrorOutOfMemory;
  ++s.mallocs;
  *p = (void*)s.next;
  s.live[s.next] = n;
  s.next += (n + 0xfffff) / 0x100000 * 0x100000;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  fake::State& s = fake::st();
  std::lock_guard<std::recursive_mutex> l(s.mu);
  if (!p) return hipSuccess;
  if (!s.live.erase((uintptr_t)p)) return hipErrorInvalidValue;
  s.freed.push_back((uintptr_t)p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void*, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyDeviceToHost) memset(dst, 0, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void*, size_t n, hipMemcpyKind k, hipStream_t q) {
  if (k == hipMemcpyDeviceToHost) memset(dst, 0, n);
  fake::push(fake::Op::Other, q);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t q) {
  fake::push(fake::Op::Other, q);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)(uintptr_t)0x200000000;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  std::lock_guard<std::recursive_mutex> l(fake::st().mu);
  *e = (hipEvent_t)malloc(16);
  fake::st().events[*e] = false;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::lock_guard<std::recursive_mutex> l(fake::st().mu);
  if (!fake::st().events.erase(e)) return hipErrorInvalidHandle;
  free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t q) {
  fake::push(fake::Op::Record, q, "", e);
  std::lock_guard<std::recursive_mutex> l(fake::st().mu);
  fake::st().events[e] = true;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  std::lock_guard<std::recursive_mutex> l(fake::st().mu);
  *ms = 1.0f;
  return fake::st().events[a] && fake::st().events[b] ? hipSuccess : hipErrorInvalidHandle;
}
hipError_t hipStreamWaitEvent(hipStream_t q, hipEvent_t e, unsigned) {
  fake::push(fake::Op::Wait, q, "", e);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t q, hipStreamCaptureStatus* c) {
  *c = fake::st().capturing.count(q) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* q, unsigned) {
  static int n = 100;
  *q = fake::stream(n++);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = nullptr;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)(uintptr_t)1;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t q) {
  fake::push(fake::Op::Launch, q, "graph");
  return hipSuccess;
}

}  // extern "C"
