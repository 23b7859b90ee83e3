// A HIP runtime without a GPU for tests of the library's host code: kernels do
// nothing but post the scalars that the solve loops wait for (struct Post),
// from values the test sets.  Loaded with RTLD_GLOBAL before the library.
//   late:  posts arrive when a stream is waited for, not when they are queued
//   fail:  so many graph launches from now on queue their work and then report
//          an error
#include <stdlib.h>
#include <string.h>

#include <deque>
#include <map>
#include <string>
#include <vector>

#include "../paper_2605_03563_amd/csrc/internal.h"

namespace {

struct Work {
  psn::Scalars* scal;
  psn::Post post;
};
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
} config;

std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::deque<Work> queue;
std::vector<Work>* recording = nullptr;
int running = 0;  // launches since a stream was last waited for

void deliver(const Work& w) {
  const unsigned seq = w.post.set ? w.post.set : w.scal->seq + 1;
  w.scal->seq = seq;
  unsigned long long* slot = w.post.mail + (seq % psn::kPostSlots) * (2 * psn::kPostMax);
  for (int i = 0; i < w.post.count; ++i) {
    unsigned long long v;
    memcpy(&v, &w.scal->v[w.post.first + i], sizeof v);
    slot[2 * i] = (unsigned long long)seq << 32 | v >> 32;
    slot[2 * i + 1] = (unsigned long long)seq << 32 | (v & 0xffffffffu);
  }
}

}  // namespace

extern "C" {

int host_late = 0, host_fail = 0, host_turns = 0;
double host_b2 = 1.0, host_r2 = 1.0;  // posted ||b||^2 and ||r||^2
double host_later = 1.0;              // ||r||^2 from post number host_turns of a solve on (0: never)

int host_running() { return running; }

static void enqueue(const Work& w) {
  ++running;
  if (!w.post.mail) return;
  static int posts = 0;
  if (w.post.set) posts = 0;
  const double r2 = host_turns && ++posts >= host_turns ? host_later : host_r2;
  for (double& v : w.scal->v) v = r2;
  w.scal->v[psn::kBnorm2] = host_b2;
  if (host_late)
    queue.push_back(w);
  else
    deliver(w);
}
static hipError_t drain() {
  for (; !queue.empty(); queue.pop_front()) deliver(queue.front());
  running = 0;
  return hipSuccess;
}

void** __hipRegisterFatBinary(const void*) { return (void**)malloc(8); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names()[f] = name;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
  config = Config{g, b, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st) {
  *g = config.grid;
  *b = config.block;
  *lds = config.lds;
  *st = config.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  const std::string& name = names()[f];
  Work w{};
  // partial, nb, nslots, scal, dst, post; partial, nb, scal, stage, post
  if (name.find("k_finish") != std::string::npos)
    w = Work{*(psn::Scalars**)args[3], *(psn::Post*)args[5]};
  else if (name.find("_scalars") != std::string::npos)
    w = Work{*(psn::Scalars**)args[2], *(psn::Post*)args[4]};
  if (recording)
    recording->push_back(w);
  else
    enqueue(w);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  recording = new std::vector<Work>;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = (hipGraph_t)recording;
  recording = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)g;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  for (const Work& w : *(std::vector<Work>*)e) enqueue(w);
  return host_fail > 0 && host_fail-- ? hipErrorUnknown : hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return drain(); }
hipError_t hipEventSynchronize(hipEvent_t) { return drain(); }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(8); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "host"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }

}  // extern "C"
