// Block ranges of the halves of attention tiles over caches read in place, on random requests (built by
// tests/test_half_tiles_host.py with g++ from plan.cpp): a half walks the blocks of its tile's range that
// start within the reach of its rows, and at least one block.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "common.h"

namespace mpic {  // (api.hip is linked for mpic_destroy and mpic_plan_destroy; nothing is launched)
hipError_t launch_assemble(int, const AssembleArgs&, const AssembleSrcTable&, hipStream_t) { return hipSuccess; }
hipError_t launch_attn_bf16(const AttnArgs&, const AssembleArgs*, const AssembleSrcTable*, const LazyRefs*, hipStream_t) { return hipSuccess; }
hipError_t launch_attn_f32(const AttnArgs&, int64_t, const LazyRefs*, hipStream_t) { return hipSuccess; }
hipError_t launch_decode(int, const DecodeArgs&, const LazyRefs*, hipStream_t) { return hipSuccess; }
hipError_t decode_static_scratch(float**, size_t*) { return hipErrorInvalidDevice; }
}  // namespace mpic

#define CHECK(...) do { if (!(__VA_ARGS__)) { std::fprintf(stderr, "check failed: %s (line %d, case %d)\n", #__VA_ARGS__, __LINE__, iter); return 1; } } while (0)

// One request per entry of `rows`: that many fresh rows behind a chunk of `len` stored ones.
bool in_halves(int hq, int hkv, int requests, int rows, int len) {
  mpic_config cfg{};
  cfg.n_q_heads = hq;
  cfg.n_kv_heads = hkv;
  cfg.head_dim = 128;
  cfg.dtype = MPIC_BF16;
  cfg.rope_theta = 1e4;
  cfg.lazy_rope = 1;
  mpic_ctx* ctx = nullptr;
  mpic_plan* p = nullptr;
  if (mpic_create(&ctx, &cfg) != MPIC_OK) return false;
  std::vector<int32_t> seg_off(1, 0);
  std::vector<mpic_segment> segs(2 * requests);
  for (int b = 0; b < requests; ++b) {
    segs[2 * b].kind = 1;
    segs[2 * b].chunk = b;
    segs[2 * b].len = len;
    segs[2 * b + 1].len = rows;
    seg_off.push_back(2 * b + 2);
  }
  const bool halves = mpic_plan_create(ctx, requests, seg_off.data(), segs.data(), 0, nullptr, nullptr, 0, &p) == MPIC_OK && p->half_tiles;
  mpic_plan_destroy(p);
  mpic_destroy(ctx);
  return halves;
}

int main() {
  {  // which launches run in halves: low tiles up to four blocks per compute unit, tall ones unless they are cut into long pieces, or very many
    const int iter = -2;
    CHECK(in_halves(32, 32, 4, 40, 400) && !in_halves(32, 32, 4, 40, 600));
    CHECK(!in_halves(32, 32, 8, 96, 5000));
    CHECK(in_halves(32, 32, 3, 240, 1000) && !in_halves(32, 32, 3, 240, 6000));
    CHECK(in_halves(32, 32, 12, 240, 3000) && !in_halves(32, 32, 30, 240, 6000));
    CHECK(!in_halves(32, 32, 14, 192, 2880));  // as many blocks as the twelve, and no padding that smaller ones would save
  }
  std::mt19937 rng(11);
  auto rnd = [&](int lo, int hi) { return lo + static_cast<int>(rng() % static_cast<unsigned>(hi - lo + 1)); };
  const int heads[][2] = {{4, 4}, {28, 4}, {32, 8}, {7, 1}, {40, 1}, {64, 8}};
  int n_shorter = 0, n_alone = 0, n_blind = 0;
  for (int iter = 0; iter < 400; ++iter) {
    mpic_config cfg{};
    cfg.n_q_heads = heads[iter % 6][0];
    cfg.n_kv_heads = heads[iter % 6][1];
    cfg.head_dim = 128;
    cfg.dtype = MPIC_BF16;
    cfg.rope_theta = 1e4;
    cfg.lazy_rope = 1;
    mpic_ctx* ctx = nullptr;
    CHECK(mpic_create(&ctx, &cfg) == MPIC_OK);
    const int B = rnd(1, 3);
    std::vector<int32_t> seg_off(1, 0), sel_off(1, 0), sel;
    std::vector<mpic_segment> segs;
    int32_t chunk = 0;
    for (int b = 0; b < B; ++b) {
      for (int i = rnd(0, 5); i > 0; --i) {
        mpic_segment s{};
        s.kind = rnd(0, 1);
        s.chunk = s.kind ? chunk++ : 0;
        s.len = s.kind ? rnd(1, iter % 5 ? 500 : 2500) : rnd(0, 90);
        s.k = rnd(0, 40);
        if (s.kind && iter % 3 == 0) {
          s.k = MPIC_K_LISTED;
          for (int32_t t = 0; t < s.len; ++t)
            if (rnd(0, 15) == 0) sel.push_back(t);
        }
        segs.push_back(s);
        sel_off.push_back(static_cast<int32_t>(sel.size()));
      }
      seg_off.push_back(static_cast<int32_t>(segs.size()));
    }
    mpic_plan* p = nullptr;
    CHECK(mpic_plan_create_selected(ctx, B, seg_off.data(), segs.data(), 8, sel_off.data(), sel.data(), nullptr, nullptr, 0, &p) == MPIC_OK);
    const int s = mpic::block_size_index(mpic::kHalfTileBlock), group = ctx->group;
    CHECK(p->lazy_half.size() == (p->half_tiles ? p->tiles.size() * 8 : 0) && p->lazy_range[s].size() == p->tiles.size() * 4);
    for (size_t i = 0; p->half_tiles && i < p->tiles.size(); ++i) {
      const mpic::AttnTile& t = p->tiles[i];
      const int32_t* r = p->lazy_range[s].data() + 4 * i;
      for (int half = 0; half < 2; ++half) {
        const int32_t* h = p->lazy_half.data() + 8 * i + 4 * half;
        const int32_t row = half * mpic::kAttnTileRows / 2;
        if (row >= t.n_rows) {
          CHECK(h[0] == 0 && h[1] == 0 && h[2] == 0 && h[3] == 0);
          n_alone += t.n_rows > 0;
          continue;
        }
        const int32_t last = t.row0 + std::min(t.n_rows, row + mpic::kAttnTileRows / 2) - 1;
        const int32_t reach = p->q_pos[p->q_off[t.req] + last / group];
        CHECK(h[0] == r[0] && h[2] == r[2] && h[1] >= h[0] && h[1] <= r[1] && h[3] >= h[2] && h[3] <= r[3]);
        CHECK(h[1] - h[0] + h[3] - h[2] >= 1);
        const mpic::KeyBlock* fresh = p->kblk[s].data() + p->kblk_first[s][t.req];
        const mpic::KeyBlock* stored = p->kblk[s].data() + p->kblk_mid[s][t.req];
        int seen = 0;
        for (int32_t k = r[0]; k < r[1]; ++k) seen += fresh[k].pos0 <= reach;
        for (int32_t k = r[2]; k < r[3]; ++k) seen += stored[k].pos0 <= reach;
        for (int32_t k = h[1]; k < r[1]; ++k) CHECK(fresh[k].pos0 > reach);
        for (int32_t k = h[3]; k < r[3]; ++k) CHECK(stored[k].pos0 > reach);
        CHECK(h[1] - h[0] + h[3] - h[2] == std::max(1, seen));
        n_shorter += h[1] < r[1] || h[3] < r[3];
        n_blind += seen == 0;
      }
    }
    mpic_plan_destroy(p);
    mpic_destroy(ctx);
  }
  const int iter = -1;
  std::printf("%d shorter, %d alone, %d blind\n", n_shorter, n_alone, n_blind);
  CHECK(n_shorter > 300 && n_alone > 100 && n_blind > 100);
  std::puts("half tiles ok");
  return 0;
}
