// fp32 selective attention of libmpic (gfx950).
//
// App. A: a_ij = exp(q_i.k_j * scale) / sum_{t<=i} exp(q_i.k_t * scale) and
// o_i = sum_{j<=i} a_ij v_j, evaluated for the rows of the recompute set only
// (Fig. 7 step 3), with "j <= i" taken by position inside the linked context.
// A workgroup owns 32 flattened rows (fresh row x query head of one kv group) of one request and
// kv head; f32_tile.h holds its work and what bounds it.
#include "common.h"
#include "f32_tile.h"

namespace mpic {
namespace {

// kLazy (lazy_rope contexts): a stored key still lacks its position shift; it is turned to its
// global position in LDS (the pair (x, y) of the key becomes (x cos - y sin, x sin + y cos)), in
// fp32, and never written back.  With refs.by_ref the stored rows are read in their caches
// instead of the context.
template <int D, bool kLazy>
__global__ __launch_bounds__(f32tile::kThreads, 2) void attn_f32_kernel(AttnArgs a, LazyRefs refs) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int lane = threadIdx.x & 63, col = lane & 31, hi = lane >> 5;
  const int group = a.n_q_heads / a.n_kv_heads;
  // workgroups of one kv head stay on one L2 domain when the heads are a multiple of eight
  const int g = static_cast<int>(blockIdx.x) % a.n_kv_heads;
  const AttnPieceF32 piece = a.pieces_f32[static_cast<int>(blockIdx.x) / a.n_kv_heads];
  const int row0 = piece.row0, n_cols = piece.n_rows;
  const int flat = row0 + min(col, n_cols - 1);
  const int64_t r = piece.q_off + flat / group;
  // fetched without a branch and first looked at behind the first keys: nothing waits for it on the way to them (152
  // tokens of 4 heads linked and attended 13.5 -> 13.4 us, one image with 32 heads 39.1 -> 38.8)
  const int row_pos = a.q_pos[r];
  const int rot_row = (a.q_rot ? a.q_rot : a.q_pos)[r];
  const int my_pos = col < n_cols ? row_pos : piece.key1 - 1;

  f32tile::Rows src{};
  src.off16 = a.kv_off16 + piece.ctx_off;
  src.k = static_cast<const char*>(a.k_ctx) + static_cast<int64_t>(g) * D * 4;
  src.v = static_cast<const char*>(a.v_ctx) + static_cast<int64_t>(g) * D * 4;
  if constexpr (kLazy) {
    src.inst = a.src_inst + piece.ctx_off;
    src.row = a.src_row + piece.ctx_off;
    src.rope_cos = a.rope_cos;
    src.rope_sin = a.rope_sin;
    src.refs = &refs;
    src.head_bytes = static_cast<int64_t>(g) * D * 4;
    src.row_bytes = static_cast<int64_t>(a.n_kv_heads) * D * 4;
    src.interleaved = a.interleaved;
  }
  auto q_row = [&](int c) __attribute__((always_inline)) {
    const int f = row0 + min(c, n_cols - 1);
    return static_cast<const char*>(a.q) + ((piece.q_off + f / group) * static_cast<int64_t>(a.n_q_heads) + g * group + f % group) * (D * 4);
  };
  auto turn = [&](float(&q)[D / 2]) __attribute__((always_inline)) {
    if (!a.q_rot) return;
    // a query that arrives without its position is turned by its position id first
    const float* ct = a.q_cos + static_cast<int64_t>(rot_row) * (D / 2);
    const float* st = a.q_sin + static_cast<int64_t>(rot_row) * (D / 2);
    if (a.interleaved) {
#pragma unroll
      for (int j = 0; j < D / 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          const int i = 2 * (2 * j + hi) + e / 2;
          const float x = q[4 * j + e], y = q[4 * j + e + 1], c = ct[i], s = st[i];
          q[4 * j + e] = x * c - y * s;
          q[4 * j + e + 1] = x * s + y * c;
        }
    } else {
#pragma unroll
      for (int j = 0; j < D / 16; ++j)  // chunk 2 j + hi and its partner half a row further
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * (2 * j + hi) + e;
          const float x = q[4 * j + e], y = q[4 * (j + D / 16) + e], c = ct[i], s = st[i];
          q[4 * j + e] = x * c - y * s;
          q[4 * (j + D / 16) + e] = x * s + y * c;
        }
    }
  };
  f32tile::attend<D, kLazy, true>(src, q_row, turn, my_pos, piece.key0, piece.key1, a.scale, lds,
                            [&](int c, int d0, const float(&o)[f32tile::Geo<D>::kPerThread], float m, float l) {
    if (c >= n_cols) return;
    const float inv = 1.f / l;
    if (piece.part >= 0) {
      // piece of a tile: a row that sees none of its keys has no weight to divide by
      const int64_t slot = (static_cast<int64_t>(piece.part) * a.n_kv_heads + g) * f32tile::kCols + c;
      float* po = a.ws_o + slot * D + d0;
#pragma unroll
      for (int i = 0; i < f32tile::Geo<D>::kPerThread; i += 4)
        *reinterpret_cast<f32x4*>(po + i) = l == 0.f ? f32x4{0} : f32x4{o[i], o[i + 1], o[i + 2], o[i + 3]} * inv;
      if (d0 == 0) a.ws_lse[slot] = l == 0.f ? -INFINITY : m * a.scale + logf(l);
      return;
    }
    const int f = row0 + c;
    const int64_t item = (piece.q_off + f / group) * static_cast<int64_t>(a.n_q_heads) + g * group + f % group;
    float* op = static_cast<float*>(a.out) + item * D + d0;
#pragma unroll
    for (int i = 0; i < f32tile::Geo<D>::kPerThread; i += 4)
      *reinterpret_cast<f32x4*>(op + i) = f32x4{o[i], o[i + 1], o[i + 2], o[i + 3]} * inv;
    if (a.lse && d0 == 0) a.lse[item] = m * a.scale + logf(l);
  });
}

// Merge the pieces of tiles that were cut along the keys: a workgroup per tile, kv head and 8 of its rows, a
// thread per four coordinates.  Bound by the way of the partial results to memory and back; they are fetched
// four pieces at a time before they are combined.
template <int D>
__global__ __launch_bounds__(2 * D) void merge_f32_kernel(AttnArgs a) {
  const AttnMerge m = a.merges[blockIdx.x];
  const int g = blockIdx.y / 4, row = blockIdx.y % 4 * 8 + threadIdx.x / (D / 4), d = threadIdx.x % (D / 4) * 4;
  if (row >= m.n_rows) return;
  const int group = a.n_q_heads / a.n_kv_heads;
  const int64_t step = static_cast<int64_t>(a.n_kv_heads) * f32tile::kCols;
  const int64_t slot0 = m.first_part * step + g * f32tile::kCols + row;
  float mx = -INFINITY, z = 0.f;
  f32x4 o = f32x4{0};
  constexpr int kDepth = 4;
  for (int p0 = 0; p0 < m.n_parts; p0 += kDepth) {
    float lse[kDepth];
    f32x4 x[kDepth];
#pragma unroll
    for (int i = 0; i < kDepth; ++i) {
      const int64_t slot = slot0 + min(p0 + i, m.n_parts - 1) * step;
      lse[i] = p0 + i < m.n_parts ? a.ws_lse[slot] : -INFINITY;
      x[i] = *reinterpret_cast<const f32x4*>(a.ws_o + slot * D + d);
    }
#pragma unroll
    for (int i = 0; i < kDepth; ++i) {
      if (lse[i] == -INFINITY) continue;  // (the first piece has a key for every row)
      const float m_new = fmaxf(mx, lse[i]);
      const float keep = expf(mx - m_new), w = expf(lse[i] - m_new);
      z = z * keep + w;
      o = o * keep + w * x[i];
      mx = m_new;
    }
  }
  const int flat = m.row0 + row;
  const int64_t item = (m.q_off + flat / group) * static_cast<int64_t>(a.n_q_heads) + g * group + flat % group;
  *reinterpret_cast<f32x4*>(static_cast<float*>(a.out) + item * D + d) = o * (1.f / z);
  if (a.lse && d == 0) a.lse[item] = mx + logf(z);
}

template <int D, bool kLazy>
hipError_t launch(const AttnArgs& a, int64_t n_pieces, const LazyRefs& refs, int dev, hipStream_t stream) {
  constexpr int kLds = f32tile::Geo<D>::kLdsBytes;
  static LdsOptIn opt_in;
  const hipError_t e = opt_in.ensure(dev, [] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(attn_f32_kernel<D, kLazy>), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  });
  if (e != hipSuccess) return e;
  const dim3 grid(static_cast<unsigned>(n_pieces) * a.n_kv_heads);
  hipLaunchKernelGGL((attn_f32_kernel<D, kLazy>), grid, dim3(f32tile::kThreads), kLds, stream, a, refs);
  if (a.n_merges > 0) hipLaunchKernelGGL((merge_f32_kernel<D>), dim3(a.n_merges, a.n_kv_heads * 4), dim3(2 * D), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

static_assert(f32tile::kCols == kAttnTileRowsF32, "tile size and kernel shape must agree");

hipError_t launch_attn_f32(const AttnArgs& a, int64_t n_pieces, const LazyRefs* lazy, hipStream_t stream) {
  if (n_pieces <= 0) return hipSuccess;
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (a.head_dim == 64)
    return lazy ? launch<64, true>(a, n_pieces, *lazy, dev, stream) : launch<64, false>(a, n_pieces, LazyRefs{}, dev, stream);
  return lazy ? launch<128, true>(a, n_pieces, *lazy, dev, stream) : launch<128, false>(a, n_pieces, LazyRefs{}, dev, stream);
}

}  // namespace mpic
