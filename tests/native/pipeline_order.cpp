// Host-only check of the order in which mpic_prefill_layers lets its launches run (built by
// tests/test_host_sanitizers.py with g++ from plan.cpp, store.cpp and the stand-ins below).  Streams and
// events are replaced by a record of what happens before what, linking and attention by what they read and
// write.  Whatever of a call's buffers overlaps, two launches of which one writes what the other touches have to be ordered as
// one mpic_assemble_kv and one mpic_selective_attn per layer order them.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>
#include <set>
#include <vector>

#include "common.h"

namespace {
struct Span {
  const char* at;
  size_t bytes;
};
struct Launch {
  int step;  // 2 * layer: linking, 2 * layer + 1: attention
  std::vector<Span> reads, writes;
  std::set<int> before;  // launches that are done when this one starts
};
std::vector<Launch> launches;
std::map<hipStream_t, std::set<int>> done_on;     // by the work enqueued on a stream so far
std::map<hipEvent_t, std::set<int>> done_at;
hipStream_t const kCaller = reinterpret_cast<hipStream_t>(16);

void enqueue(hipStream_t s, std::vector<Launch> together) {
  const std::set<int> before = done_on[s];
  for (Launch& x : together) {
    x.before = before;
    done_on[s].insert(static_cast<int>(launches.size()));
    launches.push_back(x);
  }
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n ? n : 1); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { return hipMalloc(p, n); }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new int(0)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<int*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { done_at[e] = done_on[s]; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(new int(0)); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { delete reinterpret_cast<int*>(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned int) {
  done_on[s].insert(done_at[e].begin(), done_at[e].end());
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
}

namespace {
// the buffers of the call that is being recorded, and the bytes of their rows
struct Call {
  std::vector<const void*> q, k, v;
  std::vector<void*> kc, vc, out;
  std::vector<float*> lse;
  size_t row = 0, q_row = 0, lse_row = 0;
} call;
int attended = 0;            // layers whose attention is enqueued
int carried = 0, alone = 0;  // fresh rows that went along with an attention launch, linking launches of their own
Span span(const void* p, size_t n) { return {static_cast<const char*>(p), n}; }
Launch link_of(int layer, int64_t slots, int64_t rows, bool fresh) {
  Launch x;
  x.step = 2 * layer;
  if (fresh) x.reads = {span(call.k[layer], rows * call.row), span(call.v[layer], rows * call.row)};
  x.writes = {span(call.kc[layer], slots * call.row), span(call.vc[layer], slots * call.row)};
  return x;
}
}  // namespace

namespace mpic {
int bind_device(mpic_ctx* ctx) { ctx->device = 0; return MPIC_OK; }
int next_linked = 0;  // layers whose stored rows are enqueued, in order
int assemble_parts(mpic_ctx*, mpic_plan* plan, const mpic_chunk_src*, int32_t, const void*, const void*, int64_t, void*, void*,
                   int64_t n_slots, uint32_t parts, void* stream) {
  const int layer = parts & MPIC_PART_CACHED ? next_linked++ : attended;
  ++alone;
  enqueue(static_cast<hipStream_t>(stream), {link_of(layer, n_slots, plan->n_q, parts & MPIC_PART_FRESH)});
  return MPIC_OK;
}
int attend(mpic_ctx*, mpic_plan* plan, const void*, int64_t, const void*, const void*, int64_t n_slots, double, void*, float*,
           void* stream, const NextLink* next, int32_t, const SrcRefs*) {
  const int l = attended++;
  Launch x;
  x.step = 2 * l + 1;
  x.reads = {span(call.q[l], plan->n_q * call.q_row), span(call.kc[l], n_slots * call.row), span(call.vc[l], n_slots * call.row)};
  x.writes = {span(call.out[l], plan->n_q * call.q_row)};
  if (call.lse[l]) x.writes.push_back(span(call.lse[l], plan->n_q * call.lse_row));
  std::vector<Launch> both = {x};
  if (next) {
    both.push_back(link_of(next_linked++, n_slots, plan->n_q, next->fresh_k != nullptr));
    if (next->fresh_k) *next->took_fresh = true, ++carried;
  }
  enqueue(static_cast<hipStream_t>(stream), both);
  return MPIC_OK;
}
}  // namespace mpic

extern "C" void mpic_plan_destroy(mpic_plan* plan) { delete plan; }
extern "C" void mpic_destroy(mpic_ctx* ctx) {
  if (ctx->link_stream) (void)hipStreamDestroy(ctx->link_stream);
  for (hipEvent_t ev : ctx->ev_layer) (void)hipEventDestroy(ev);
  delete ctx;
}

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); std::exit(1); } } while (0)

namespace {
bool overlap(const std::vector<Span>& x, const std::vector<Span>& y) {
  for (const Span& a : x)
    for (const Span& b : y)
      if (a.at < b.at + b.bytes && b.at < a.at + a.bytes) return true;
  return false;
}
// Every two launches of different steps that meet in a buffer run in the order of the steps.
bool in_order() {
  for (size_t i = 0; i < launches.size(); ++i)
    for (size_t j = 0; j < launches.size(); ++j) {
      const Launch &a = launches[i], &b = launches[j];
      if (a.step >= b.step) continue;
      if (!overlap(a.writes, b.writes) && !overlap(a.writes, b.reads) && !overlap(a.reads, b.writes)) continue;
      if (!b.before.count(static_cast<int>(i))) {
        std::fprintf(stderr, "layer %d %s does not wait for layer %d %s\n", b.step / 2, b.step & 1 ? "attention" : "linking", a.step / 2,
                     a.step & 1 ? "attention" : "linking");
        return false;
      }
    }
  return true;
}

constexpr int kLayers = 4;

struct Setup {
  mpic_ctx* ctx = nullptr;
  mpic_store* st = nullptr;
  mpic_plan* plan = nullptr;
  uint64_t id = 7;
  size_t ctx_bytes = 0, fresh_bytes = 0, q_bytes = 0, lse_bytes = 0;
  std::vector<char> memory;

  Setup(int dtype, int tier, bool fits_tail) {
    mpic_config cfg{};
    cfg.n_q_heads = fits_tail ? 8 : 4;
    cfg.n_kv_heads = 4;
    cfg.head_dim = 128;
    cfg.dtype = dtype;
    cfg.rope_theta = 1e4;
    CHECK(mpic_create(&ctx, &cfg) == MPIC_OK);
    CHECK(mpic_store_create(ctx, kLayers, nullptr, 1, &st) == MPIC_OK);
    const int len = 300;
    const size_t elem = dtype == MPIC_F32 ? 4 : 2;
    call = Call{};
    call.row = cfg.n_kv_heads * cfg.head_dim * elem;
    call.q_row = cfg.n_q_heads * cfg.head_dim * elem;
    call.lse_row = cfg.n_q_heads * sizeof(float);
    std::vector<char> cache(kLayers * len * call.row);
    CHECK(mpic_store_put(st, id, len, cache.data(), cache.data(), tier, -1) == MPIC_OK);
    mpic_segment segs[2] = {};
    segs[0].len = 20;
    segs[1].kind = 1;
    segs[1].len = len;
    segs[1].k = 4;
    const int32_t seg_off[2] = {0, 2};
    CHECK(mpic_plan_create(ctx, 1, seg_off, segs, 4, nullptr, nullptr, 0, &plan) == MPIC_OK);
    ctx_bytes = plan->n_ctx * call.row;
    fresh_bytes = plan->n_q * call.row;
    q_bytes = plan->n_q * call.q_row;
    lse_bytes = plan->n_q * call.lse_row;
    memory.resize(kLayers * (2 * ctx_bytes + 2 * fresh_bytes + 2 * q_bytes + lse_bytes + 7 * 64) + 64);
  }
  ~Setup() {
    mpic_plan_destroy(plan);
    mpic_store_destroy(st);
    mpic_destroy(ctx);
  }
  void distinct() {  // a buffer of its own for everything
    char* p = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(memory.data()) + 63) / 64 * 64);
    auto take = [&](size_t n) { char* x = p; p += (n + 63) / 64 * 64; return x; };
    call.q.clear(), call.k.clear(), call.v.clear(), call.kc.clear(), call.vc.clear(), call.out.clear(), call.lse.clear();
    for (int l = 0; l < kLayers; ++l) {
      call.q.push_back(take(q_bytes));
      call.k.push_back(take(fresh_bytes));
      call.v.push_back(take(fresh_bytes));
      call.kc.push_back(take(ctx_bytes));
      call.vc.push_back(take(ctx_bytes));
      call.out.push_back(take(q_bytes));
      call.lse.push_back(reinterpret_cast<float*>(take(lse_bytes)));
    }
  }
  bool ordered() {
    launches.clear(), done_on.clear(), done_at.clear();
    attended = carried = alone = mpic::next_linked = 0;
    CHECK(mpic_prefill_layers(ctx, plan, st, &id, 1, kLayers, call.q.data(), call.k.data(), call.v.data(), plan->n_q, call.kc.data(),
                              call.vc.data(), plan->n_ctx, 0.1, call.out.data(), call.lse.data(), kCaller, nullptr) == MPIC_OK);
    CHECK(attended == kLayers && mpic::next_linked == kLayers);
    return in_order();
  }
};
}  // namespace

int main() {
  std::mt19937 rng(11);
  for (int dtype : {MPIC_BF16, MPIC_F32})
    for (int tier : {MPIC_TIER_HBM, MPIC_TIER_HOST})
      for (bool fits : {true, false}) {
        Setup s(dtype, tier, fits);
        const bool tail = dtype == MPIC_BF16 && tier == MPIC_TIER_HBM && mpic::link_fits_attention_tail(s.ctx, s.plan);
        s.distinct();
        CHECK(s.ordered());
        CHECK(carried == (tail ? kLayers - 1 : 0) && (!tail || alone == 1));
        // one overlap at a time, every kind with the next layer's and with a later layer's context or fresh rows
        for (int to = 1; to < kLayers; ++to)
          for (int what = 0; what < 5; ++what)
            for (int where = 0; where < 4; ++where) {
              s.distinct();
              char* at = where == 0   ? static_cast<char*>(call.kc[to])
                         : where == 1 ? static_cast<char*>(call.vc[to]) + call.row
                         : where == 2 ? static_cast<char*>(const_cast<void*>(call.k[to]))
                                      : static_cast<char*>(const_cast<void*>(call.v[to]));
              if (what == 0) call.q[0] = at;
              if (what == 1) call.k[0] = at;
              if (what == 2) call.out[0] = at;
              if (what == 3) call.lse[0] = reinterpret_cast<float*>(at);
              if (what == 4 && where < 2) call.kc[0] = where ? static_cast<char*>(call.kc[to]) + 2 * call.row : at;
              if (!s.ordered()) {
                std::fprintf(stderr, "dtype %d tier %d: buffer %d of layer 0 in buffer %d of layer %d\n", dtype, tier, what, where, to);
                return 1;
              }
            }
        // buffers all over the place
        for (int trial = 0; trial < 300; ++trial) {
          s.distinct();
          char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(s.memory.data()) + 63) / 64 * 64);
          for (int n = 1 + static_cast<int>(rng() % 6); n > 0; --n) {
            char* at = base + rng() % ((s.memory.size() - s.ctx_bytes - s.q_bytes) / 64) * 64;
            const int l = static_cast<int>(rng() % kLayers);
            switch (rng() % 6) {
              case 0: call.q[l] = at; break;
              case 1: call.k[l] = at; break;
              case 2: call.kc[l] = at; break;
              case 3: call.vc[l] = at; break;
              case 4: call.out[l] = at; break;
              default: call.lse[l] = reinterpret_cast<float*>(at);
            }
          }
          if (!s.ordered()) {
            std::fprintf(stderr, "dtype %d tier %d trial %d\n", dtype, tier, trial);
            return 1;
          }
        }
      }
  std::puts("pipeline order ok");
  return 0;
}
