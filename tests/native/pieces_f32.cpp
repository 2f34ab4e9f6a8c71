// Work items of the fp32 attention on random requests (built by tests/test_pieces_f32_host.py with g++
// from plan.cpp): tiles cover every row once, the pieces of a tile cover its keys once, and every
// partial result is merged once.
#include <cstdint>
#include <cstdio>
#include <map>
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

int main() {
  std::mt19937 rng(7);
  auto rnd = [&](int lo, int hi) { return lo + static_cast<int>(rng() % static_cast<unsigned>(hi - lo + 1)); };
  const int heads[][2] = {{4, 4}, {32, 32}, {6, 2}, {7, 1}, {40, 1}, {12, 12}};
  int n_cut = 0, n_whole = 0;
  for (int iter = 0; iter < 600; ++iter) {
    mpic_config cfg{};
    cfg.n_q_heads = heads[iter % 6][0];
    cfg.n_kv_heads = heads[iter % 6][1];
    cfg.head_dim = iter % 2 ? 64 : 128;
    cfg.dtype = MPIC_F32;
    cfg.rope_theta = 1e4;
    mpic_ctx* ctx = nullptr;
    CHECK(mpic_create(&ctx, &cfg) == MPIC_OK);
    const int B = rnd(1, 3);
    std::vector<int32_t> seg_off(1, 0);
    std::vector<mpic_segment> segs;
    int32_t chunk = 0;
    for (int b = 0; b < B; ++b) {
      for (int i = rnd(0, 4); i > 0; --i) {
        mpic_segment s{};
        s.kind = rnd(0, 1);
        s.chunk = s.kind ? chunk++ : 0;
        s.len = s.kind ? rnd(1, iter % 5 ? 400 : 2500) : rnd(0, 90);
        s.k = rnd(0, 40);
        segs.push_back(s);
      }
      seg_off.push_back(static_cast<int32_t>(segs.size()));
    }
    mpic_plan* p = nullptr;
    CHECK(mpic_plan_create(ctx, B, seg_off.data(), segs.data(), 8, nullptr, nullptr, 0, &p) == MPIC_OK);
    const int group = ctx->group;
    std::map<std::pair<int, int>, mpic::AttnPieceF32> tiles;
    int64_t rows = 0;
    for (const auto& t : p->tiles_f32) {
      CHECK(t.n_rows >= 1 && t.n_rows <= mpic::kAttnTileRowsF32 && t.row0 % mpic::kAttnTileRowsF32 == 0);
      CHECK(t.key0 == 0 && t.part == -1 && t.q_off == p->q_off[t.req] && t.ctx_off == p->ctx_off[t.req]);
      CHECK(t.key1 == p->q_pos[t.q_off + (t.row0 + t.n_rows - 1) / group] + 1);
      CHECK(tiles.emplace(std::make_pair(t.req, t.row0), t).second);
      rows += t.n_rows;
    }
    CHECK(rows == p->n_q * group);
    if (p->pieces_f32.empty()) {
      CHECK(p->merges_f32.empty() && p->n_parts_f32 == 0);
      n_whole += !tiles.empty();
    } else {
      ++n_cut;
      std::map<std::pair<int, int>, std::map<int, mpic::AttnPieceF32>> of_tile;  // by first key
      for (const auto& x : p->pieces_f32) CHECK(of_tile[{x.req, x.row0}].emplace(x.key0, x).second);
      CHECK(of_tile.size() == tiles.size());
      std::vector<int> merged(p->n_parts_f32, 0);
      for (const auto& m : p->merges_f32) {
        const auto& pieces = of_tile.at({m.req, m.row0});
        CHECK(static_cast<int>(pieces.size()) == m.n_parts && m.n_parts > 1 && m.q_off == p->q_off[m.req]);
        CHECK(m.n_rows == tiles.at({m.req, m.row0}).n_rows);
        int part = m.first_part;
        for (const auto& x : pieces) {  // in key order
          CHECK(x.second.part == part);
          CHECK(part < p->n_parts_f32);
          ++merged[part++];
        }
      }
      for (int n : merged) CHECK(n == 1);
      for (const auto& t : of_tile) {
        int32_t key = 0;
        for (const auto& x : t.second) {
          CHECK(x.second.key0 == key && x.second.key1 > key && x.second.key0 % 32 == 0);
          CHECK((x.second.part >= 0) == (t.second.size() > 1) && x.second.n_rows == tiles.at(t.first).n_rows);
          key = x.second.key1;
        }
        CHECK(key == tiles.at(t.first).key1);
      }
    }
    mpic_plan_destroy(p);
    mpic_destroy(ctx);
  }
  const int iter = -1;
  CHECK(n_cut > 100 && n_whole > 50);
  std::puts("fp32 pieces ok");
  return 0;
}
