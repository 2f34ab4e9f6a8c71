// Host-only exercise of the pool of plan blocks (csrc/plan_blocks.h), built by
// tests/test_host_sanitizers.py with g++.  Streams and events are stand-ins with a clock each, so
// that work can be left pending; the pool must never hand out a block that pending work reads, and
// must keep the runtime's malloc and free out of the usual ways in which plans come and go.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <set>
#include <vector>

#include "plan_blocks.h"

namespace {
struct Stream {
  long enqueued = 0, finished = 0;
  bool capturing = false, destroyed = false;
};
struct Event {
  Stream* stream = nullptr;
  long at = 0;
};
Stream null_stream;
bool bad_handle = false;
Stream* of(hipStream_t s) {
  Stream* x = s ? reinterpret_cast<Stream*>(s) : &null_stream;
  if (x->destroyed) bad_handle = true;
  return x;
}
hipStream_t handle(Stream* s) { return s == &null_stream ? nullptr : reinterpret_cast<hipStream_t>(s); }
int n_events = 0;
}  // namespace

extern "C" {
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = of(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) { return of(s)->finished == of(s)->enqueued ? hipSuccess : hipErrorNotReady; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(new Event());
  ++n_events;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<Event*>(e);
  --n_events;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (of(s)->capturing) return hipErrorStreamCaptureUnsupported;
  *reinterpret_cast<Event*>(e) = Event{of(s), of(s)->enqueued};
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  const Event* x = reinterpret_cast<Event*>(e);
  return !x->stream || x->stream->finished >= x->at ? hipSuccess : hipErrorNotReady;
}
}

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); std::exit(1); } } while (0)

namespace {
// Plans as the library makes, uses and destroys them.
struct Plan {
  void* block = nullptr;
  size_t bytes = 0;
  mpic::PlanUse use;
};
struct Runtime {
  mpic::SpareBlocks pool;
  int mallocs = 0, frees = 0;
  std::map<void*, std::vector<Event>> readers;  // work that reads a block

  Plan first_use(size_t need, Stream* s) {
    Plan p;
    p.block = pool.take(need, &p.bytes, handle(s));
    if (p.block) {
      CHECK(p.bytes >= need);
      for (const Event& w : readers[p.block]) CHECK(w.stream->finished >= w.at);
      readers[p.block].clear();
    } else {
      p.bytes = mpic::SpareBlocks::size_for(need);
      p.block = std::malloc(1);
      ++mallocs;
    }
    run(&p, s);
    return p;
  }
  void run(Plan* p, Stream* s) {
    p->use.add(handle(s));
    if (!s->capturing) readers[p->block].push_back(Event{s, ++s->enqueued});
  }
  void release(void* block) {  // hipFree: waits for the GPU
    ++frees;
    readers.erase(block);
    std::free(block);
  }
  void destroy(Plan* p) {
    void* replaced = nullptr;
    if (!pool.give(p->block, p->bytes, p->use, &replaced)) release(p->block);
    if (replaced) release(replaced);
  }
  ~Runtime() {
    pool.close([&](void* b) { release(b); });
  }
};
void wait(Stream* s) { s->finished = s->enqueued; }
}  // namespace

int main() {
  {  // a request is finished and its plan destroyed before the next one is made
    Runtime rt;
    for (int i = 0; i < 50; ++i) {
      Plan p = rt.first_use(100000, &null_stream);
      rt.run(&p, &null_stream);
      wait(&null_stream);
      rt.destroy(&p);
    }
    CHECK(rt.mallocs == 1 && rt.frees == 0);
  }
  for (const bool lagging : {false, true}) {  // the next plan is made first; the GPU is up to two requests behind
    Runtime rt;
    Plan last = rt.first_use(100000, &null_stream);
    for (int i = 0; i < 50; ++i) {
      Plan p = rt.first_use(100000 + 200 * (i % 7), &null_stream);
      rt.destroy(&last);
      last = p;
      null_stream.finished = lagging ? null_stream.enqueued - 2 : null_stream.enqueued;
    }
    CHECK(rt.mallocs <= 4 && rt.frees == 0);
    wait(&null_stream);
    rt.destroy(&last);
  }
  {  // a request that is also worked on by the library's own stream (layer pipeline)
    Runtime rt;
    Stream caller, link;
    rt.pool.own(handle(&link));
    for (int i = 0; i < 50; ++i) {
      Plan p = rt.first_use(100000, i % 2 ? &link : &caller);
      rt.run(&p, &link);
      rt.run(&p, &caller);
      if (i % 3 == 0) wait(&link);
      wait(&caller);
      rt.destroy(&p);
      wait(&link);
    }
    CHECK(rt.mallocs <= 3 && rt.frees == 0);
  }
  {  // a conversation whose plans grow, after a warm-up on short ones
    Runtime rt;
    int n = 0;
    for (size_t need = 70000; need < (size_t{12} << 20); need += need / 30, ++n) {
      Plan p = rt.first_use(need, &null_stream);
      wait(&null_stream);
      rt.destroy(&p);
    }
    CHECK(n > 140 && rt.mallocs <= 17 && rt.frees <= 17);
    const int mallocs = rt.mallocs, frees = rt.frees;
    for (int i = 0; i < 100; ++i) {
      Plan p = rt.first_use((size_t{11} << 20) + 1000 * i, &null_stream);
      wait(&null_stream);
      rt.destroy(&p);
    }
    CHECK(rt.mallocs == mallocs && rt.frees == frees);
  }
  {  // streams that go with their requests: their handles are not touched, later plans find room
    Runtime rt;
    std::vector<Stream> gone(4);
    for (Stream& s : gone) {
      Plan p = rt.first_use(100000, &s);
      wait(&s);
      s.destroyed = true;
      rt.destroy(&p);
    }
    CHECK(rt.frees == 0);
    const int mallocs = rt.mallocs;
    for (int i = 0; i < 20; ++i) {
      Plan p = rt.first_use(100000, &null_stream);
      wait(&null_stream);
      rt.destroy(&p);
    }
    CHECK(rt.mallocs == mallocs + 1 && rt.frees == 1 && !bad_handle);
  }
  for (size_t need = 1; need <= mpic::SpareBlocks::kMaxBytes; need += need / 7 + 1) {
    const size_t size = mpic::SpareBlocks::size_for(need);
    CHECK(size >= need && size <= mpic::SpareBlocks::kMaxBytes && (size <= need / 2 * 3 + 2 || size == size_t{64} << 10));
  }
  {  // not followed: under capture, on the per-thread stream, on too many streams, too large, pool closed
    Runtime rt;
    Stream s[4];
    Plan p = rt.first_use(1000, &s[0]);
    s[0].capturing = true;
    rt.run(&p, &s[0]);
    s[0].capturing = false;
    rt.run(&p, &s[0]);
    wait(&s[0]);
    rt.destroy(&p);
    CHECK(rt.frees == 1);
    p = rt.first_use(1000, &s[0]);
    p.use.add(hipStreamPerThread);
    wait(&s[0]);
    rt.destroy(&p);
    CHECK(rt.frees == 2);
    p = rt.first_use(1000, &s[0]);
    for (Stream& x : s) rt.run(&p, &x);
    for (Stream& x : s) wait(&x);
    rt.destroy(&p);
    CHECK(rt.frees == 3);
    p = rt.first_use(mpic::SpareBlocks::kMaxBytes + 1, &s[0]);
    CHECK(p.bytes == mpic::SpareBlocks::kMaxBytes + 1);
    rt.destroy(&p);
    CHECK(rt.frees == 4);
    p = rt.first_use(1000, &s[0]);
    rt.pool.close([&](void* b) { rt.release(b); });
    rt.destroy(&p);
    CHECK(rt.frees == 5);
  }
  {  // anything goes: what is handed out is never read by pending work (checked in first_use)
    std::mt19937 rng(7);
    Runtime rt;
    Stream s[4];
    rt.pool.own(handle(&s[3]));
    std::vector<Plan> alive;
    for (int i = 0; i < 200000; ++i) {
      Stream* on = &s[rng() % 4];
      switch (rng() % 5) {
        case 0: alive.push_back(rt.first_use(1000 << rng() % 10, on)); break;
        case 1: if (!alive.empty()) rt.run(&alive[rng() % alive.size()], on); break;
        case 2:
          if (!alive.empty()) {
            std::swap(alive[rng() % alive.size()], alive.back());
            rt.destroy(&alive.back());
            alive.pop_back();
          }
          break;
        case 3: if (on->finished < on->enqueued) ++on->finished; break;
        default: if (rng() % 8 == 0) wait(on); else if (rng() % 8 == 0) on->capturing = !on->capturing;
      }
    }
    CHECK(rt.mallocs > 100);
    for (Plan& p : alive) rt.destroy(&p);
  }
  CHECK(n_events == 0 && !bad_handle);
  std::puts("plan blocks ok");
  return 0;
}
