// Host-only exercise of the scratch memory behind the entry points (built by
// tests/test_host_sanitizers.py with g++ from plan.cpp, api.hip and the stand-ins below): who
// allocates it, what happens when it cannot be had, which calls share it.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <thread>
#include <vector>

#include "common.h"

// ---- stand-ins for the HIP runtime: host memory, a limit on it, streams that may be captured ----
namespace {
size_t in_use = 0, limit = SIZE_MAX;
std::map<void*, size_t> sizes;
int n_syncs = 0;
struct Stream { bool capturing = false; };
bool capturing_any = false;
Stream null_stream;
Stream per_thread;
Stream* of(hipStream_t s) { return s == hipStreamPerThread ? &per_thread : s ? reinterpret_cast<Stream*>(s) : &null_stream; }
}  // namespace
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (capturing_any) return hipErrorStreamCaptureUnsupported;
  if (in_use + n > limit) return hipErrorOutOfMemory;
  *p = std::malloc(n ? n : 1);
  sizes[*p] = n;
  in_use += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  in_use -= sizes.at(p);
  sizes.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new int(0)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<int*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(new Stream()); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { delete of(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = of(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { ++n_syncs; return capturing_any ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
}

namespace mpic {
AttnArgs last_attn;
DecodeArgs last_decode;
AssembleArgs last_assemble;
hipError_t launch_assemble(int, const AssembleArgs& a, const AssembleSrcTable&, hipStream_t) { last_assemble = a; return hipSuccess; }
hipError_t launch_attn_bf16(const AttnArgs& a, const AssembleArgs*, const AssembleSrcTable*, const LazyRefs*, hipStream_t) {
  last_attn = a;
  return hipSuccess;
}
hipError_t launch_attn_f32(const AttnArgs& a, int64_t, const LazyRefs*, hipStream_t) { last_attn = a; return hipSuccess; }
hipError_t launch_decode(int, const DecodeArgs& a, const LazyRefs*, hipStream_t) { last_decode = a; return hipSuccess; }
hipError_t decode_static_scratch(float**, size_t*) { return hipErrorInvalidDevice; }
}  // namespace mpic

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); std::exit(1); } } while (0)

namespace {
alignas(16) char any[16];  // stands for every data buffer: the launches are stand-ins
mpic_ctx* context(int dtype) {
  mpic_config cfg{};
  cfg.n_q_heads = 8;
  cfg.n_kv_heads = 8;
  cfg.head_dim = 128;
  cfg.dtype = dtype;
  cfg.rope_theta = 1e4;
  mpic_ctx* ctx = nullptr;
  CHECK(mpic_create(&ctx, &cfg) == MPIC_OK);
  return ctx;
}
mpic_plan* plan_of(mpic_ctx* ctx, int len) {  // one request of text
  const int32_t seg_off[2] = {0, 1};
  mpic_segment seg{};
  seg.len = len;
  mpic_plan* p = nullptr;
  CHECK(mpic_plan_create(ctx, 1, seg_off, &seg, 0, nullptr, nullptr, 0, &p) == MPIC_OK);
  return p;
}
int assemble(mpic_ctx* c, mpic_plan* p, Stream* s) {
  return mpic_assemble_kv(c, p, nullptr, 0, any, any, p->n_q, any, any, p->n_ctx, s);
}
int attend(mpic_ctx* c, mpic_plan* p, Stream* s) {
  return mpic_selective_attn(c, p, any, p->n_q, any, any, p->n_ctx, 0.1, any, nullptr, s);
}
int decode(mpic_ctx* c, mpic_plan* p, Stream* s) {
  return mpic_decode_attn(c, p, any, nullptr, nullptr, any, any, p->n_ctx, 0.1, any, nullptr, s);
}
size_t ws_of(const mpic_plan* p) { return static_cast<size_t>(p->n_parts) * mpic::kAttnTileRows * 129 * sizeof(float); }
void capture(Stream* s, bool on) { s->capturing = capturing_any = on; }
}  // namespace

int main() {
  const size_t mb = size_t{1} << 20;
  Stream s[7];
  {  // without room for the workspace a plan can be linked and decoded; only its attention fails
    mpic_ctx* c = context(MPIC_BF16);
    mpic_plan* p = plan_of(c, 3000);
    CHECK(p->n_parts > 0 && ws_of(p) > 4 * mb);
    limit = in_use + 2 * mb;
    CHECK(assemble(c, p, &s[0]) == MPIC_OK);
    CHECK(decode(c, p, &s[0]) == MPIC_OK);
    CHECK(attend(c, p, &s[0]) == MPIC_ERR_OOM);
    limit = SIZE_MAX;
    CHECK(attend(c, p, &s[0]) == MPIC_OK);
    // a larger plan finds room for its workspace only if the old one goes, once the GPU is idle
    mpic_plan* q = plan_of(c, 9000);
    CHECK(ws_of(q) > ws_of(p));
    limit = in_use + ws_of(q) - ws_of(p) + mb;
    const int syncs = n_syncs;
    CHECK(assemble(c, q, &s[0]) == MPIC_OK && n_syncs == syncs);
    CHECK(attend(c, q, &s[0]) == MPIC_OK && n_syncs == syncs + 1);
    limit = SIZE_MAX;
    mpic_plan_destroy(p);
    mpic_plan_destroy(q);
    mpic_destroy(c);
    CHECK(in_use == 0);
  }
  {  // linking on the default stream leaves a workspace too
    mpic_ctx* c = context(MPIC_BF16);
    mpic_plan* p = plan_of(c, 3000);
    CHECK(assemble(c, p, nullptr) == MPIC_OK);
    capture(&s[5], true);
    CHECK(attend(c, p, &s[5]) == MPIC_OK);
    capture(&s[5], false);
    mpic_plan_destroy(p);
    mpic_destroy(c);
    CHECK(in_use == 0);
  }
  {  // streams do not meet in a workspace, capture finds the one that linking left; what is outgrown stays
    mpic_ctx* c = context(MPIC_BF16);
    mpic_plan* p = plan_of(c, 3000);
    CHECK(assemble(c, p, &s[0]) == MPIC_OK);
    capture(&s[5], true);
    CHECK(attend(c, p, &s[5]) == MPIC_OK);
    capture(&s[5], false);
    const float* captured = mpic::last_attn.ws_o;
    CHECK(attend(c, p, &s[0]) == MPIC_OK && mpic::last_attn.ws_o == captured);
    std::vector<const float*> of_stream;
    const int syncs = n_syncs;
    for (int i = 0; i < 4; ++i) {
      CHECK(attend(c, p, &s[i]) == MPIC_OK);
      for (const float* w : of_stream) CHECK(mpic::last_attn.ws_o != w);
      of_stream.push_back(mpic::last_attn.ws_o);
    }
    for (int i = 0; i < 4; ++i) CHECK(attend(c, p, &s[i]) == MPIC_OK && mpic::last_attn.ws_o == of_stream[i]);
    CHECK(n_syncs == syncs);
    CHECK(attend(c, p, &s[4]) == MPIC_OK && n_syncs == syncs + 1);  // a fifth stream
    mpic_plan* q = plan_of(c, 9000);
    CHECK(assemble(c, q, &s[3]) == MPIC_OK);
    capture(&s[3], true);
    CHECK(attend(c, q, &s[3]) == MPIC_OK && mpic::last_attn.ws_o != of_stream[3]);
    capture(&s[3], false);
    CHECK(sizes.count(const_cast<float*>(of_stream[3])) == 1);
    mpic_plan_destroy(q);
    mpic_plan_destroy(p);
    mpic_destroy(c);
    CHECK(in_use == 0);
  }
  for (int dtype : {MPIC_BF16, MPIC_F32}) {  // hipStreamPerThread is another stream in every thread, each with its own workspace
    mpic_ctx* c = context(dtype);
    mpic_plan* p = plan_of(c, dtype == MPIC_BF16 ? 3000 : 700);
    Stream* mine = reinterpret_cast<Stream*>(hipStreamPerThread);
    const auto ws = [&](Stream* x) {
      CHECK(attend(c, p, x) == MPIC_OK && mpic::last_attn.ws_o);
      return mpic::last_attn.ws_o;
    };
    const int syncs = n_syncs;
    const float *first = ws(&s[0]), *here = ws(mine), *there = nullptr;
    std::thread([&] { there = ws(mine); }).join();
    CHECK(first != here && there != here && there != first && ws(mine) == here && ws(&s[0]) == first && n_syncs == syncs);
    mpic_plan_destroy(p);
    mpic_destroy(c);
    CHECK(in_use == 0);
  }
  {  // fp32: tiles are cut only where the stream itself has room for their partial results, and whole otherwise
    mpic_ctx* c = context(MPIC_F32);
    mpic_plan* p = plan_of(c, 700);
    CHECK(p->n_parts_f32 > 0);
    const auto cut = [&] {  // pieces, merge list and workspace go together
      const mpic::AttnArgs& a = mpic::last_attn;
      CHECK(a.pieces_f32 == (a.ws_o ? p->dev.pieces_f32 : p->dev.tiles_f32));
      CHECK(a.n_merges == (a.ws_o ? static_cast<int32_t>(p->merges_f32.size()) : 0));
      return a.ws_o != nullptr;
    };
    limit = in_use + mb / 2;  // the plan's tables fit, the workspace does not
    CHECK(assemble(c, p, &s[0]) == MPIC_OK && attend(c, p, &s[0]) == MPIC_OK && !cut());
    limit = SIZE_MAX;
    CHECK(attend(c, p, &s[0]) == MPIC_OK && cut());
    std::vector<const float*> of_stream = {mpic::last_attn.ws_o};
    // a capture may run at any time: it takes no workspace, of its own stream or of another
    for (Stream* x : {&s[0], &s[5]}) {
      capture(x, true);
      CHECK(attend(c, p, x) == MPIC_OK && !cut());
      capture(x, false);
    }
    for (int i = 1; i < 4; ++i) {
      CHECK(attend(c, p, &s[i]) == MPIC_OK && cut());
      for (const float* w : of_stream) CHECK(mpic::last_attn.ws_o != w);
      of_stream.push_back(mpic::last_attn.ws_o);
    }
    const int syncs = n_syncs;
    CHECK(attend(c, p, &s[4]) == MPIC_OK && !cut() && n_syncs == syncs);  // a fifth stream waits for nothing
    CHECK(attend(c, p, &s[1]) == MPIC_OK && mpic::last_attn.ws_o == of_stream[1]);
    mpic_plan_destroy(p);
    mpic_destroy(c);
    CHECK(in_use == 0);
  }
  {  // fp32 plans that are not cut take no workspace; decode steps of one batch size stay valid as contexts grow
    mpic_ctx* c = context(MPIC_F32);
    mpic_plan *p = plan_of(c, 200), *q = plan_of(c, 5000);
    CHECK(assemble(c, p, &s[0]) == MPIC_OK && assemble(c, q, &s[0]) == MPIC_OK);
    CHECK(p->n_parts_f32 == 0 && q->n_parts_f32 == 0 && attend(c, q, &s[0]) == MPIC_OK);
    for (const mpic::Scratch& w : c->attn_ws) CHECK(!w.ptr);
    capture(&s[1], true);  // no step before has left any room
    CHECK(decode(c, q, &s[1]) == MPIC_OK && mpic::last_decode.n_splits == 1 && mpic::last_decode.keys_per_split == 5000);
    capture(&s[1], false);
    CHECK(decode(c, p, &s[0]) == MPIC_OK && mpic::last_decode.n_splits == 1);
    float* const first = mpic::last_decode.ws_o;  // as a captured step holds it
    capture(&s[1], true);
    CHECK(decode(c, q, &s[1]) == MPIC_OK && mpic::last_decode.n_splits == 1 && mpic::last_decode.keys_per_split == 5000);
    CHECK(mpic::last_decode.ws_o == first);
    capture(&s[1], false);
    const int syncs = n_syncs;
    CHECK(decode(c, q, &s[0]) == MPIC_OK && mpic::last_decode.n_splits > 1 && mpic::last_decode.ws_o != first);
    CHECK(sizes.count(first) == 1 && n_syncs == syncs);
    mpic_plan_destroy(p);
    mpic_plan_destroy(q);
    mpic_destroy(c);
    CHECK(in_use == 0);
  }
  {  // a decode step whose keys are not split needs no memory, captured or not; a split one that finds none fails
    mpic_ctx* c = context(MPIC_BF16);
    mpic_plan *p = plan_of(c, 200), *q = plan_of(c, 600);
    CHECK(assemble(c, p, &s[0]) == MPIC_OK && assemble(c, q, &s[0]) == MPIC_OK);
    capture(&s[1], true);
    CHECK(decode(c, p, &s[1]) == MPIC_OK && mpic::last_decode.n_splits == 1);
    capture(&s[1], false);
    limit = in_use;
    CHECK(decode(c, p, &s[0]) == MPIC_OK && mpic::last_decode.n_splits == 1);
    CHECK(decode(c, q, &s[0]) == MPIC_ERR_OOM);
    limit = SIZE_MAX;
    CHECK(!c->decode_ws.ptr);
    mpic_plan_destroy(p);
    mpic_plan_destroy(q);
    mpic_destroy(c);
    CHECK(in_use == 0);
  }
  {  // the linking kernel is told how far its contexts reach, except from 4 GiB on, which offsets of 32 bits do not cover
    for (const int dtype : {MPIC_BF16, MPIC_F32})
      for (const int past : {0, 1}) {
        mpic_config cfg{8, 8, 128, dtype, 1e4, 0, 16, 0, 0};
        mpic_ctx* c = nullptr;
        CHECK(mpic_create(&c, &cfg) == MPIC_OK);
        const int64_t row = dtype == MPIC_F32 ? 4096 : 2048, pages = (int64_t{1} << 32) / row / 16 - 1 + past;
        const int32_t seg_off[2] = {0, 1}, table_off[2] = {0, 1}, table[1] = {static_cast<int32_t>(pages - 1)};
        mpic_segment seg{};
        seg.len = 16;
        mpic_plan* p = nullptr;
        CHECK(mpic_plan_create(c, 1, seg_off, &seg, 0, table, table_off, pages, &p) == MPIC_OK);
        CHECK(mpic_assemble_kv(c, p, nullptr, 0, any, any, p->n_q, any, any, pages * 16, &s[0]) == MPIC_OK);
        CHECK(mpic::last_assemble.ctx_bytes == (past ? 0 : pages * 16 * row));
        mpic_plan_destroy(p);
        mpic_destroy(c);
      }
    CHECK(in_use == 0);
  }
  std::puts("scratch ok");
  return 0;
}
