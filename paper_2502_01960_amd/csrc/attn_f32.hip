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
  // workgroups of one kv head stay on one L2 domain when the heads are a multiple of eight; the
  // last rows of the batch, which see most keys, come first
  const int g = static_cast<int>(blockIdx.x) % a.n_kv_heads;
  int tile = static_cast<int>(gridDim.x / a.n_kv_heads) - 1 - static_cast<int>(blockIdx.x) / a.n_kv_heads;
  int b = 0, rows = 0;
  for (;; ++b) {
    rows = (a.q_off[b + 1] - a.q_off[b]) * group;
    const int n = (rows + f32tile::kCols - 1) / f32tile::kCols;
    if (tile < n) break;
    tile -= n;
  }
  const int row0 = tile * f32tile::kCols;
  const int n_cols = min(rows - row0, f32tile::kCols);
  const int n_keys = a.q_pos[a.q_off[b] + (row0 + n_cols - 1) / group] + 1;
  const int flat = row0 + min(col, n_cols - 1);
  const int64_t r = a.q_off[b] + flat / group;
  const int my_pos = col < n_cols ? a.q_pos[r] : n_keys - 1;

  float q[D / 2];
  f32tile::load_query<D>(static_cast<const float*>(a.q) + (r * a.n_q_heads + g * group + flat % group) * D, hi, q);
  if (a.q_rot) {
    // a query that arrives without its position is turned by its position id first
    const float* ct = a.q_cos + static_cast<int64_t>(a.q_rot[r]) * (D / 2);
    const float* st = a.q_sin + static_cast<int64_t>(a.q_rot[r]) * (D / 2);
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
  }

  f32tile::Rows src{};
  src.off16 = a.kv_off16 + a.ctx_off[b];
  src.k = static_cast<const char*>(a.k_ctx) + static_cast<int64_t>(g) * D * 4;
  src.v = static_cast<const char*>(a.v_ctx) + static_cast<int64_t>(g) * D * 4;
  if constexpr (kLazy) {
    src.inst = a.src_inst + a.ctx_off[b];
    src.row = a.src_row + a.ctx_off[b];
    src.rope_cos = a.rope_cos;
    src.rope_sin = a.rope_sin;
    src.refs = &refs;
    src.head_bytes = static_cast<int64_t>(g) * D * 4;
    src.row_bytes = static_cast<int64_t>(a.n_kv_heads) * D * 4;
    src.interleaved = a.interleaved;
  }
  f32tile::attend<D, kLazy>(src, q, my_pos, 0, n_keys, a.scale, lds,
                            [&](int c, int d0, const float(&o)[f32tile::Geo<D>::kPerThread], float m, float l) {
    if (c >= n_cols) return;
    const int f = row0 + c;
    const int64_t item = (a.q_off[b] + f / group) * static_cast<int64_t>(a.n_q_heads) + g * group + f % group;
    const float inv = 1.f / l;
    float* op = static_cast<float*>(a.out) + item * D + d0;
#pragma unroll
    for (int i = 0; i < f32tile::Geo<D>::kPerThread; i += 4)
      *reinterpret_cast<f32x4*>(op + i) = f32x4{o[i], o[i + 1], o[i + 2], o[i + 3]} * inv;
    if (a.lse && d0 == 0) a.lse[item] = m * a.scale + logf(l);
  });
}

template <int D, bool kLazy>
hipError_t launch(const AttnArgs& a, int64_t n_tiles, const LazyRefs& refs, int dev, hipStream_t stream) {
  constexpr int kLds = f32tile::Geo<D>::kLdsBytes;
  static LdsOptIn opt_in;
  const hipError_t e = opt_in.ensure(dev, [] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(attn_f32_kernel<D, kLazy>), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  });
  if (e != hipSuccess) return e;
  const dim3 grid(static_cast<unsigned>(n_tiles) * a.n_kv_heads);
  hipLaunchKernelGGL((attn_f32_kernel<D, kLazy>), grid, dim3(f32tile::kThreads), kLds, stream, a, refs);
  return hipGetLastError();
}

}  // namespace

static_assert(f32tile::kCols == kAttnTileRowsF32, "tile size and kernel shape must agree");

hipError_t launch_attn_f32(const AttnArgs& a, int64_t n_tiles, const LazyRefs* lazy, hipStream_t stream) {
  if (n_tiles <= 0) return hipSuccess;
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (a.head_dim == 64)
    return lazy ? launch<64, true>(a, n_tiles, *lazy, dev, stream) : launch<64, false>(a, n_tiles, LazyRefs{}, dev, stream);
  return lazy ? launch<128, true>(a, n_tiles, *lazy, dev, stream) : launch<128, false>(a, n_tiles, LazyRefs{}, dev, stream);
}

}  // namespace mpic
