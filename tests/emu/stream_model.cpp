// Host model of a HIP stream for the library's host code: the calls of the HIP
// runtime and the kernel launches that sv_api.cpp, sv_batch.cpp and
// sv_exec.cpp make are replaced by functions that queue what they read and
// write.  Nothing queued has run until something waits for it; buffers that
// queued work still uses may be neither freed nor rewritten, and a call that
// promises a finished buffer has to leave none of its work queued.
//
//   stream_model <scenario>    exits 0, or 1 with what went wrong
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "sv_host.h"

namespace {

struct Span {
  const unsigned char* at;
  size_t bytes;
};
struct Work {
  const char* what;
  std::vector<Span> uses;
};
std::vector<Work> queue;   // everything enqueued, in order (one stream)
size_t finished = 0;       // queue[0 .. finished) has run
std::map<void*, size_t> allocs;
std::map<hipEvent_t, size_t> events;
std::vector<size_t> pinned_sizes;
int faults = 0;
int fail_launch = -1;  // the batched launch (counted from 0) that fails
int batch_launches = 0;
uint64_t batch_tiles = 0;

void fault(const std::string& s) {
  std::printf("%s\n", s.c_str());
  ++faults;
}

size_t block_size(const void* p) {
  auto it = allocs.find(const_cast<void*>(p));
  return it == allocs.end() ? 0 : it->second;
}

// `what` needs that no queued work uses the span any more.
void must_be_idle(const char* what, const void* p, size_t bytes) {
  const unsigned char* a = (const unsigned char*)p;
  for (size_t i = finished; i < queue.size(); ++i)
    for (const Span& s : queue[i].uses)
      if (a < s.at + s.bytes && s.at < a + bytes) {
        fault(std::string(what) + " while " + queue[i].what + " may still use the buffer");
        return;
      }
}

void enqueue(const char* what, std::vector<Span> uses) { queue.push_back({what, std::move(uses)}); }
Span span(const void* p, size_t bytes) { return {(const unsigned char*)p, bytes}; }

}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  allocs[*p] = n;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  pinned_sizes.push_back(n);
  return hipMalloc(p, n);
}
hipError_t hipFree(void* p) {
  if (p) must_be_idle("hipFree", p, block_size(p));
  std::free(p);
  allocs.erase(p);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  // the caller has just filled `src`
  must_be_idle("a host buffer was rewritten", src, n);
  std::memcpy(dst, src, n);
  enqueue("a copy", {span(dst, n), span(src, n)});
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free((void*)e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  events[e] = queue.size();
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (events[e] > finished) finished = events[e];
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  finished = queue.size();
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "model"; }
}

namespace sv {
hipError_t launch_sweep(sv_dtype, void*, int, const SweepArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_probs(sv_dtype, const void*, int, const int*, int, double*, void*, hipStream_t) { return hipSuccess; }
size_t probs_scratch_bytes(int, int, const int*) { return 0; }
size_t static_scratch_bytes() { return 0; }
hipError_t static_scratch(int, void** p) {
  *p = nullptr;
  return hipErrorInvalidValue;
}
hipError_t launch_init_basis(sv_dtype, void*, int, uint64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_copy_bytes(void*, const void*, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_dense_kq(sv_dtype, void*, int, int, const int*, const void*, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_matrix_pass(int, void*, int, int, const PassDescDev*, int, int, const PassStageDev*, const void*,
                              hipStream_t) {
  return hipSuccess;
}
hipError_t launch_pass(sv_dtype, void*, int, int, const PassDescDev* passes, int pass, const PassStageDev*,
                       const PassItemDev*, const void*, const void*, bool, PassMatrix, hipStream_t) {
  enqueue("a pass", {span(passes + pass, sizeof(PassDescDev))});
  return hipSuccess;
}
hipError_t launch_stage_frags(PassStageDev* stages, const uint32_t* list, int count, const void* pool, void* frags,
                              hipStream_t) {
  enqueue("the fragment build", {span(list, count * sizeof(uint32_t)), span(stages, sizeof(PassStageDev)),
                                 span(pool, 16), span(frags, (size_t)count * kStageFragBytes)});
  return hipSuccess;
}
hipError_t launch_pass_batch(sv_dtype, const BatchItemDev* items, int count, uint64_t tiles, int, bool, PassMatrix,
                             hipStream_t) {
  if (batch_launches++ == fail_launch) return hipErrorInvalidValue;
  for (int i = 1; i < count; ++i)
    if (items[i].tile_begin <= items[i - 1].tile_begin || items[i].tile_begin >= tiles) fault("tile ranges out of order");
  if (items[0].tile_begin != 0) fault("the first item does not start at tile 0");
  batch_tiles += tiles;
  enqueue("a batched pass", {span(items, count * sizeof(BatchItemDev))});
  return hipSuccess;
}
}  // namespace sv

namespace {

sv_gate gate(int kind, std::vector<int> q, double theta = 0.0) {
  sv_gate g{};
  g.kind = kind;
  g.nq = (int)q.size();
  for (int i = 0; i < SV_MAX_GATE_QUBITS; ++i) g.q[i] = i < g.nq ? q[i] : -1;
  g.theta = theta;
  return g;
}

// A plan with matrix fragments: QFT-like blocks in tile passes, or fused ops
// in matrix passes.
sv_plan* plan(int n, int mode, int max_fuse) {
  std::vector<sv_gate> gs;
  for (int rep = 0; rep < 3; ++rep)
    for (int q = n - 1; q >= 0; --q) {
      gs.push_back(gate(SV_G_H, {q}));
      for (int c = q - 1; c >= 0; --c) gs.push_back(gate(SV_G_CPHASE, {c, q}, 0.1 + c));
    }
  sv_opts o;
  sv_default_opts(&o);
  o.mode = mode;
  o.max_fuse_qubits = max_fuse;
  sv_plan* p = nullptr;
  if (sv_fuse(n, SV_C64, gs.data(), gs.size(), &o, &p) != SV_OK) {
    fault(std::string("plan: ") + sv_last_error());
    std::exit(1);
  }
  return p;
}

void expect(sv_status st, sv_status want) {
  if (st != want) fault(std::string("status ") + std::to_string(st) + ": " + sv_last_error());
}

// A program in the caller's buffer is destroyed without having been run: its
// own work on the buffer has to be over by then.
void scenario_program() {
  for (int mode : {(int)SV_MODE_PASS, (int)SV_MODE_MATRIX}) {
    sv_plan* p = plan(13, mode, 5);
    size_t bytes = 0;
    expect(sv_program_bytes(p, &bytes), SV_OK);
    void* buf = nullptr;
    (void)hipMalloc(&buf, bytes);
    sv_program* prog = nullptr;
    expect(sv_program_create(p, buf, bytes, nullptr, &prog), SV_OK);
    size_t builds = 0;
    for (const Work& w : queue) builds += std::strcmp(w.what, "the fragment build") == 0;
    if (!builds) fault("the plan has no matrix fragments");
    expect(sv_program_destroy(prog), SV_OK);
    must_be_idle("sv_program_destroy returned", buf, bytes);
    (void)hipStreamSynchronize(nullptr);
    (void)hipFree(buf);
    sv_plan_destroy(p);
    queue.clear();
    finished = 0;
  }
}

// A step of several launches fails after its first: the descriptors it has
// enqueued are still read when its slot comes round again.
void scenario_batcher() {
  const int n = 13;
  sv_plan* plans[2] = {plan(n, SV_MODE_PASS, 5), plan(n, SV_MODE_MATRIX, 5)};  // tile stages, matrix stages
  sv_program* progs[2];
  sv_state* states[2];
  for (int i = 0; i < 2; ++i) {
    expect(sv_program_create(plans[i], nullptr, 0, nullptr, &progs[i]), SV_OK);
    expect(sv_create(n, SV_C64, nullptr, nullptr, SV_NO_INIT, &states[i]), SV_OK);
  }
  sv_batcher* b = nullptr;
  expect(sv_batcher_create(nullptr, &b), SV_OK);
  int32_t pass[2] = {0, -1};
  for (int32_t k = 0, kind, ops, local, stages; pass[1] < 0; ++k) {
    expect(sv_plan_pass_info(plans[1], (size_t)k, &kind, &ops, &local, &stages), SV_OK);
    if (faults) return;
    if (kind == sv::PASS_MATRIX) pass[1] = k;
  }
  for (int failing = 0; failing < 2; ++failing) {
    batch_launches = 0;
    fail_launch = failing;
    expect(sv_batcher_run(b, 2, states, progs, pass), SV_ERR_DEVICE);
    fail_launch = -1;
    for (int i = 0; i < 9; ++i) expect(sv_batcher_run(b, 2, states, progs, pass), SV_OK);
    if (batch_launches != failing + 1 + 18) fault("a step is not two launches");
  }
  expect(sv_batcher_destroy(b), SV_OK);
  for (int i = 0; i < 2; ++i) {
    expect(sv_program_destroy(progs[i]), SV_OK);
    expect(sv_destroy(states[i]), SV_OK);
    sv_plan_destroy(plans[i]);
  }
}

// Tile passes with and without matrix stages run in one launch.
void scenario_launches() {
  for (int n : {13, 22}) {  // one tile, 512 tiles
    sv_gate g[2] = {gate(SV_G_RY, {3}, 0.2), gate(SV_G_RX, {8}, 0.4)};
    sv_opts o;
    sv_default_opts(&o);
    o.mode = SV_MODE_PASS;
    sv_plan* plans[2] = {plan(n, SV_MODE_PASS, 5), nullptr};  // on the matrix cores, on the VALU
    expect(sv_fuse(n, SV_C64, g, 2, &o, &plans[1]), SV_OK);
    sv_program* progs[2];
    sv_state* states[2];
    for (int i = 0; i < 2; ++i) {
      expect(sv_program_create(plans[i], nullptr, 0, nullptr, &progs[i]), SV_OK);
      expect(sv_create(n, SV_C64, nullptr, nullptr, SV_NO_INIT, &states[i]), SV_OK);
    }
    sv_batcher* b = nullptr;
    expect(sv_batcher_create(nullptr, &b), SV_OK);
    const int32_t pass[2] = {0, 0};
    batch_launches = 0;
    batch_tiles = 0;
    expect(sv_batcher_run(b, 2, states, progs, pass), SV_OK);
    if (batch_launches != 1) fault("N = " + std::to_string(n) + ": " + std::to_string(batch_launches) + " launches");
    if (batch_tiles != (2ull << (n - 13))) fault("N = " + std::to_string(n) + ": " + std::to_string(batch_tiles) + " tiles");
    expect(sv_batcher_destroy(b), SV_OK);
    for (int i = 0; i < 2; ++i) {
      expect(sv_program_destroy(progs[i]), SV_OK);
      expect(sv_destroy(states[i]), SV_OK);
      sv_plan_destroy(plans[i]);
    }
  }
}

// Pinned staging memory holds what is staged, not the fragments that are built
// on the device behind it.
void scenario_staging() {
  sv_state* st = nullptr;
  expect(sv_create(13, SV_C64, nullptr, nullptr, SV_NO_INIT, &st), SV_OK);
  for (int mode : {(int)SV_MODE_PASS, (int)SV_MODE_MATRIX, (int)SV_MODE_PASS}) {
    sv_plan* p = plan(13, mode, 5);
    sv::PackedPlan pk;
    expect(sv::pack_plan(p, &pk), SV_OK);
    pinned_sizes.clear();
    queue.clear();
    finished = 0;
    expect(sv_apply_plan(st, p), SV_OK);
    for (size_t n : pinned_sizes)
      if (n > 65536 && n >= 2 * pk.host.size())
        fault("staging buffer of " + std::to_string(n) + " bytes for " + std::to_string(pk.host.size()));
    // the device buffer holds the image and the fragments
    for (const Work& w : queue)
      for (const Span& s : w.uses) {
        bool inside = false;
        for (const auto& a : allocs)
          inside = inside || (s.at >= (unsigned char*)a.first && s.at + s.bytes <= (unsigned char*)a.first + a.second);
        if (!inside) fault(std::string(w.what) + " uses memory outside the buffers");
      }
    (void)hipStreamSynchronize(nullptr);
    sv_plan_destroy(p);
  }
  expect(sv_destroy(st), SV_OK);
}

}  // namespace

int main(int argc, char** argv) {
  const std::string s = argc > 1 ? argv[1] : "";
  if (s == "program") scenario_program();
  else if (s == "batcher") scenario_batcher();
  else if (s == "launches") scenario_launches();
  else if (s == "staging") scenario_staging();
  else fault("unknown scenario");
  return faults ? 1 : 0;
}
