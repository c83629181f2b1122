// The library's calls on a HIP runtime that runs nothing: every runtime function the library uses is defined
// here (the program's own definitions come before the runtime library's) and logged, one line per call, with
// kernels by their names.  No GPU is touched; device pointers are never read.
//
//   calls CALL R L sigma_z sigma_dl pixel n_y n_z n plan [; R L ... ]     (a batch: several geometries)
//
// CALL: iterate, denominators, loglik, value, noalloc, batch (eager), graph (created, launched, destroyed), mixed
// (eager, graph created, eager, graph launched and destroyed), threads (two threads, each eager on its own stream).
#include <cxxabi.h>
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <chrono>
#include <map>
#include <string>
#include <thread>
#include <vector>

#include "jpet.h"

static std::map<const void*, std::string>& names() {  // (filled before this program's own initialisers run)
  static std::map<const void*, std::string> m;
  return m;
}
static std::string name_of(const void* f) {
  auto it = names().find(f);
  if (it == names().end()) return "unknown";
  int bad = 0;
  char* d = abi::__cxa_demangle(it->second.c_str(), nullptr, nullptr, &bad);
  std::string s = d ? d : it->second;
  free(d);
  for (const char* cut : {"void ", "jpet::", "(anonymous namespace)::"})
    for (size_t at; (at = s.find(cut)) != std::string::npos;) s.erase(at, strlen(cut));
  s = s.substr(0, s.find('('));
  for (size_t at; (at = s.find(' ')) != std::string::npos;) s.erase(at, 1);
  return s;
}
static std::atomic<int> ids{0};
static thread_local int me = 0;  // the thread's number, in the log of records and waits
static std::atomic<bool> slow{false};
static void* fresh() { return (void*)(size_t)(++ids * 16); }
static long id(const void* p) { return (long)((size_t)p / 16); }
static thread_local dim3 cfg_g, cfg_b;
static thread_local size_t cfg_s;
static thread_local hipStream_t cfg_st;

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* x;
  return &x;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  cfg_g = g, cfg_b = b, cfg_s = s, cfg_st = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  *g = cfg_g, *b = cfg_b, *s = cfg_s, *st = cfg_st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t lds, hipStream_t st) {
  printf("launch %s grid %u %u block %u lds %zu stream %ld\n", name_of(f).c_str(), g.x, g.y, b.x, lds, id(st));
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int v) {
  printf("limit %s lds %d\n", f ? name_of(f).c_str() : "null", v);
  return f ? hipSuccess : hipErrorInvalidDeviceFunction;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)0x100000;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void*, size_t n, hipMemcpyKind, hipStream_t) {
  memset(d, 0, n);
  *(unsigned char*)d = 77;  // a batch's instance: so many items
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)fresh();
  printf("stream+ %ld\n", id(*s));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  printf("stream- %ld\n", id(s));
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)fresh();
  printf("event+ %ld\n", id(*e));
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  printf("event- %ld\n", id(e));
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  printf("record %ld stream %ld thread %d\n", id(e), id(s), me);
  if (slow) std::this_thread::sleep_for(std::chrono::milliseconds(1));  // (lets the other thread come between)
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  printf("wait %ld stream %ld thread %d\n", id(e), id(s), me);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  printf("capture+ stream %ld\n", id(s));
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  *g = (hipGraph_t)fresh();
  printf("capture- stream %ld\n", id(s));
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)fresh();
  printf("instantiate %ld\n", id(*e));
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  printf("exec- %ld\n", id(e));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  printf("graph %ld stream %ld\n", id(e), id(s));
  return hipSuccess;
}
}

int main(int argc, char** argv) {
  const std::string call = argv[1];
  std::vector<jpet_instance> inst;
  float* const fake = (float*)0x100000;
  for (int a = 2; a + 8 < argc; a += 10) {
    jpet_instance in;
    memset(&in, 0, sizeof(in));
    jpet_geometry& g = in.g;
    g.R = atof(argv[a]), g.L = atof(argv[a + 1]), g.sigma_z = atof(argv[a + 2]), g.sigma_dl = atof(argv[a + 3]);
    g.pixel = atof(argv[a + 4]), g.n_y = atoi(argv[a + 5]), g.n_z = atoi(argv[a + 6]);
    in.n = atoll(argv[a + 7]), g.plan = atoi(argv[a + 8]);
    in.events = in.rho = fake;
    inst.push_back(in);
  }
  auto result = [](const char* what, int rc) {
    printf("rc %s %d\n", what, rc);
    return rc;
  };
  jpet_instance& one = inst[0];
  size_t bytes = 0;
  if (call == "batch" || call == "graph") {
    const int count = (int)inst.size();
    if (result("size", jpet_mlem_batched_workspace_size(inst.data(), count, &bytes))) return 0;
    result("prepare", jpet_mlem_batched_prepare(inst.data(), count, fake, bytes, nullptr));
    if (call == "batch") {
      result("iterate", jpet_mlem_batched_iterate(inst.data(), count, 2, fake, bytes, JPET_WS_PREPARED, nullptr, nullptr));
    } else {
      jpet_batched_graph* gr = nullptr;
      if (result("create", jpet_mlem_batched_graph_create(inst.data(), count, 2, fake, bytes, JPET_WS_PREPARED, nullptr, &gr)))
        return 0;
      result("launch", jpet_mlem_batched_graph_launch(gr, nullptr));
      result("destroy", jpet_mlem_batched_graph_destroy(gr));
    }
  } else if (call == "mixed") {
    const int count = (int)inst.size();
    if (result("size", jpet_mlem_batched_workspace_size(inst.data(), count, &bytes))) return 0;
    jpet_batched_graph* gr = nullptr;
    result("iterate", jpet_mlem_batched_iterate(inst.data(), count, 2, fake, bytes, 0, nullptr, nullptr));
    if (result("create", jpet_mlem_batched_graph_create(inst.data(), count, 2, fake, bytes, 0, nullptr, &gr))) return 0;
    result("again", jpet_mlem_batched_iterate(inst.data(), count, 2, fake, bytes, 0, nullptr, nullptr));
    result("launch", jpet_mlem_batched_graph_launch(gr, nullptr));
    result("destroy", jpet_mlem_batched_graph_destroy(gr));
  } else if (call == "threads") {
    const int count = (int)inst.size();
    if (result("size", jpet_mlem_batched_workspace_size(inst.data(), count, &bytes))) return 0;
    slow = true;
    std::vector<std::thread> team;
    for (int k = 1; k <= 2; ++k)
      team.emplace_back([&, k] {
        me = k;
        jpet_mlem_batched_iterate(inst.data(), count, 20, fake, bytes, 0, nullptr, (hipStream_t)(size_t)(16000 * k));
      });
    for (std::thread& t : team) t.join();
  } else if (call == "iterate") {
    if (result("size", jpet_mlem_workspace_size(&one.g, one.n, &bytes))) return 0;
    result("iterate", jpet_mlem_iterate(&one.g, fake, one.n, nullptr, fake, 2, fake, bytes, 0, nullptr, nullptr));
  } else if (call == "denominators") {
    if (result("size", jpet_mlem_workspace_size(&one.g, one.n, &bytes))) return 0;
    result("denominators", jpet_mlem_denominators(&one.g, fake, one.n, fake, fake, fake, bytes, 0, nullptr, nullptr));
  } else if (call == "loglik" || call == "value") {
    if (result("size", jpet_loglik_workspace_size(&one.g, nullptr, one.n, &bytes))) return 0;
    const bool value = call == "value";
    result("loglik", jpet_loglik_grad(&one.g, nullptr, fake, one.n, nullptr, fake, (double*)fake, value ? nullptr : fake, fake,
                                      fake, bytes, value ? JPET_LOGLIK_VALUE_ONLY : 0, nullptr, nullptr));
  } else if (call == "noalloc") {
    result("noalloc", jpet_mlem_iterate_noalloc(&one.g, fake, one.n, nullptr, fake, 2, 0, nullptr, nullptr));
  }
  return 0;
}
