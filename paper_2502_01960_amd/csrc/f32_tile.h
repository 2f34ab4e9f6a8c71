// One tile of fp32 attention on the matrix cores, shared by the fp32 prefill and decode kernels.
//
// App. A in plain fp32: 32 queries of one (request, kv head) attend to a range of positions of
// the request.  Bound by the fp32 matrix rate (v_mfma_f32_32x32x2_f32, 256 flop per cycle and
// compute unit) for prefill rows and by the stream of rows for decode rows.
//
// Split.  The eight wavefronts of a workgroup take the 32-key blocks of the range in turn, each
// with its own running softmax, and merge through LDS at the end: a small request (one block per
// wavefront) then takes the time of one block instead of that of the whole range, and nothing
// inside the loop waits for another wavefront.
//
// Both products are computed transposed (a query is a lane column, softmax statistics are per-lane
// scalars), with the lane layout A[i][k]: lane i + 32 k, B[k][j]: lane j + 32 k, C[i][j]: lane
// j + 32 ((i / 4) % 2), register (i / 8) * 4 + i % 4:
//   S^T[key][query] = K . Q^T   the two halves of a wavefront contract 16-byte chunks of a row in
//                               turn, so a lane's operand is a 16-byte LDS read of its key's row.
//                               Key rows are staged by direct global->LDS loads; chunk c of row i
//                               lies at chunk c ^ (i & 15), which makes the reads conflict-free.
//   O^T[d][query] = V^T . P^T   step r contracts keys (r/4)*8 + r%4 and +4, which is where register
//                               r of S^T already lies; row index i of block db is coordinate
//                               (D/32) i + db, so a lane's operands of all blocks are one vector
//                               load of a value row -- straight from memory, without LDS.
// The value rows of a block arrive while its keys are multiplied, the keys of the next block while
// this one is normalised and multiplied with the values.
//
// Error against float64.  Most of it is the rounding of the logits, a sum of D terms: even and odd
// chunks have an accumulator each.  With one for all of them the outputs had 0.95 to 1.23 times the error of
// plain fp32 loops over the keys, with two 0.69 to 0.96 of it (contexts of 80 to 2.6K tokens, prefill
// and decode; one image of 576 tokens with 32 heads, link + attend, 55.5 -> 56.9 us).  scale * log2(e) is held in two parts, since its
// rounding shifts the exponents of all keys the same way, and the weights are summed in fours:
// log-sum-exp of that image 1.07 -> 0.81 of the error of plain loops.
#pragma once

#include "common.h"
#include "wave_ops.h"

namespace mpic {
namespace f32tile {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kKeys = 32;  // keys per block
constexpr int kCols = 32;  // queries per tile

template <int D>
struct Geo {
  static constexpr int kChunks = D / 4;               // 16-byte chunks of a row
  static constexpr int kArea = kKeys * D * 4;         // staged key block of one wavefront
  static constexpr int kLoads = kArea / 1024;         // direct loads per block
  static constexpr int kBlocks = D / 32;              // 32-row blocks of O^T
  static constexpr int kPerThread = D / (kThreads / kCols);  // coordinates a thread merges
  static constexpr int kQuery = kWaves * kArea + 2 * kWaves * kCols * 4;  // the staged queries
  static constexpr int kLdsBytes = kQuery + kArea;
  static_assert(kCols * D * 4 == kArea, "a wavefront's partial result takes the place of its key block");
};

// Where the rows of one (request, kv head) are: every position in the context buffers, or (kLazy)
// stored keys still without their shift, possibly in their caches.
struct Rows {
  const uint32_t* off16;  // context row offsets of the request's positions, 16-byte units
  const char* k;          // context base + this head's offset inside a row
  const char* v;
  // lazy_rope contexts
  const int32_t* inst;    // chunk instance of every position, -1 = fresh row
  const int32_t* row;     // row inside that instance's cache
  const float* rope_cos;
  const float* rope_sin;
  const LazyRefs* refs;   // by_ref: stored rows are read at refs->k / refs->v
  int64_t row_bytes;
  int64_t head_bytes;
  int interleaved;
};

__device__ inline const char* from_lane(const char* p, int lane) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __shfl(static_cast<uint32_t>(u), lane), hi = __shfl(static_cast<uint32_t>(u >> 32), lane);
  return reinterpret_cast<const char*>(static_cast<uint64_t>(hi) << 32 | lo);
}

// The value again, in a form whose derived addresses the compiler does not keep across the loop
// (it would hold some 60 registers of them, and spill).
__device__ inline int here(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// q_row(i): where the query of column i lies.  It is held as q[4 j + e] = coordinate 4 (2 j + lane / 32) + e of
// column lane % 32; turn(q) may rotate it first.  my_pos: last position the column sees, key0 .. key1 - 1:
// the range.  emit(column, first coordinate, values, reference maximum of the raw logits, denominator) is called
// once per thread and column.
//
// The eight wavefronts have the same queries.  kStagedQ: they come through LDS, behind the first keys.  (Fetched by
// each wavefront from memory, 16 bytes of 64 rows at a time and before anything else: 149 rows over 693 keys with
// 32 heads 29.2 us instead of 26.5, uncut 41.0 instead of 38.3.)  Otherwise every wavefront fetches them itself, with its first
// row offsets: the way through LDS and its barrier are longer than that for the few short rows of a decode step with heads
// of 64 (843 keys with 4 heads 13.4 us through LDS, 13.1 so; with 32 heads of 128 through LDS 27.7, so 28.8).
template <int D, bool kLazy, bool kStagedQ, typename QRow, typename Turn, typename Emit>
__device__ __forceinline__ void attend(const Rows& src, QRow&& q_row, Turn&& turn, int my_pos, int key0, int key1, float scale,
                                       char* lds, Emit&& emit) {
  using G = Geo<D>;
  typedef float vrow __attribute__((ext_vector_type(G::kBlocks)));
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, col = lane & 31, hi = lane >> 5;
  char* area = lds + wave * G::kArea;
  const uint32_t area_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(MPIC_LDS_PTR(char, area)));
  // weight of a raw logit t = s - reference <= 0: exp2(t * (c + c_lo)), c + c_lo = scale * log2(e).
  // c lies below the product, so that c_lo is positive and t = -infinity gives -infinity in both terms.
  float c = scale * 1.4426950216293335f, c_lo = fmaf(scale, 1.4426950216293335f, -c) + scale * 1.9259629891e-8f;
  if (c_lo <= 0.f && c > 1e-36f) {
    const float below = __uint_as_float(__float_as_uint(c) - 1);
    c_lo += c - below;
    c = below;
  }
  c = fmaxf(c, 1e-37f);  // (0 * -infinity is no number)
  c_lo = fmaxf(c_lo, 1e-37f);
  auto weight = [&](float t) __attribute__((always_inline)) { return __builtin_amdgcn_exp2f(fmaf(t, c, t * c_lo)); };

  int lo_pos = kStagedQ ? 0 : wave_min_i32(my_pos);  // no column ends before this position

  // addresses of the key and value row that lane `lane % 32` stands for, and its rotary table row
  const char* kp = nullptr;
  const char* vp = nullptr;
  int inst = -1;
  auto locate = [&](int j0) __attribute__((always_inline)) {
    const int j = min(j0 + col, key1 - 1);  // past the range: its last row again (masked)
    const int64_t off = static_cast<int64_t>(src.off16[j]) << 4;
    kp = src.k + off;
    vp = src.v + off;
    if constexpr (kLazy) {
      inst = src.inst[j];
      if (inst >= 0 && src.refs->by_ref) {
        const int64_t at = src.row[j] * src.row_bytes + src.head_bytes;
        kp = static_cast<const char*>(src.refs->k[inst]) + at;
        vp = static_cast<const char*>(src.refs->v[inst]) + at;
      }
    }
  };
  auto stage_keys = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < G::kLoads; ++p) {
      const int ln = here(lane);
      const int r = (ln + 64 * p) / G::kChunks;
      const int ch = (ln % G::kChunks) ^ (r & 15);
      load_to_lds_16B(from_lane(kp, r) + ch * 16, area_addr + p * 1024);
      if (p % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // few addresses in registers at a time
    }
  };

  float m_run = -INFINITY, l_run = 0.f;
  f32x16 acc_o[G::kBlocks];
#pragma unroll
  for (int i = 0; i < G::kBlocks; ++i) acc_o[i] = f32x16{0};

  float q[D / 2];
  if constexpr (!kStagedQ) {
    const f32x4* row = reinterpret_cast<const f32x4*>(q_row(col)) + hi;
#pragma unroll
    for (int j = 0; j < G::kChunks / 2; ++j) {
      const f32x4 x = row[2 * j];
#pragma unroll
      for (int e = 0; e < 4; ++e) q[4 * j + e] = x[e];
    }
  }
  const int n_blk = (key1 - key0 + kKeys - 1) / kKeys;
  locate(key0 + wave * kKeys);  // (for wavefronts without a block too: no branch, and with it no wait of its own)
  MPIC_WAIT_VMCNT(0);  // ordinary loads first: from here on the counter is managed by hand
  __builtin_amdgcn_sched_barrier(0);
  if (wave < n_blk) stage_keys();
  if constexpr (kStagedQ) {
    char* area_q = lds + G::kQuery;
    const uint32_t area_q_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(MPIC_LDS_PTR(char, area_q)));
#pragma unroll
    for (int i = 0; i < G::kLoads / kWaves; ++i) {
      const int p = wave + i * kWaves, r = (lane + 64 * p) / G::kChunks;
      load_to_lds_16B(q_row(r) + ((lane % G::kChunks) ^ (r & 15)) * 16, area_q_addr + p * 1024);
    }
    lo_pos = __builtin_amdgcn_readfirstlane(wave_min_i32(my_pos));
    MPIC_WAIT_VMCNT(0);
    asm volatile("" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int j = 0; j < G::kChunks / 2; ++j) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(area_q + col * (D * 4) + (((2 * j + hi) ^ (col & 15)) << 4));
#pragma unroll
      for (int e = 0; e < 4; ++e) q[4 * j + e] = x[e];
    }
  }
  turn(q);
  if constexpr (kStagedQ) __builtin_amdgcn_sched_barrier(0);
  for (int t = wave; t < n_blk; t += kWaves) {
    const int j0 = key0 + t * kKeys;
    MPIC_WAIT_VMCNT(0);  // this block's keys have landed
    asm volatile("" ::: "memory");
    vrow v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      v[r] = *reinterpret_cast<const vrow*>(from_lane(vp, (r >> 2) * 8 + here(hi) * 4 + (r & 3)) + col * (G::kBlocks * 4));
      if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kLazy) {
      // stored keys are turned to their position where they lie, a row per lane and half the chunks per half
      if (inst >= 0) {
        const float* ct = src.rope_cos + static_cast<int64_t>(inst) * (D / 2);
        const float* st = src.rope_sin + static_cast<int64_t>(inst) * (D / 2);
        auto chunk = [&](int ch) { return reinterpret_cast<f32x4*>(area + col * (D * 4) + ((ch ^ (col & 15)) << 4)); };
        if (src.interleaved) {
          for (int ch = hi; ch < G::kChunks; ch += 2) {
            const f32x4 x = *chunk(ch);
            const float c0 = ct[2 * ch], s0 = st[2 * ch], c1 = ct[2 * ch + 1], s1 = st[2 * ch + 1];
            *chunk(ch) = f32x4{x[0] * c0 - x[1] * s0, x[0] * s0 + x[1] * c0, x[2] * c1 - x[3] * s1, x[2] * s1 + x[3] * c1};
          }
        } else {
          for (int ch = hi; ch < G::kChunks / 2; ch += 2) {
            const f32x4 x = *chunk(ch), y = *chunk(ch + G::kChunks / 2);
            const f32x4 cc = *reinterpret_cast<const f32x4*>(ct + 4 * ch), ss = *reinterpret_cast<const f32x4*>(st + 4 * ch);
            *chunk(ch) = x * cc - y * ss;
            *chunk(ch + G::kChunks / 2) = x * ss + y * cc;
          }
        }
      }
      asm volatile("" ::: "memory");
    }
    f32x16 s = f32x16{0}, s_odd = f32x16{0};
    // (key operands are read two steps ahead; the scheduling barriers keep the compiler from reading
    // all of them first, which costs 64 registers and spills)
    auto key_chunk = [&](int j) __attribute__((always_inline)) {
      return *reinterpret_cast<const f32x4*>(area + here(col) * (D * 4) + (((2 * j + hi) ^ (here(col) & 15)) << 4));
    };
    f32x4 kf[2] = {key_chunk(0), key_chunk(1)};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < G::kChunks / 2; ++j) {
      const f32x4 k = kf[j & 1];
      if (j + 2 < G::kChunks / 2) kf[j & 1] = key_chunk(j + 2);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (j & 1)
          s_odd = __builtin_amdgcn_mfma_f32_32x32x2f32(k[e], q[4 * j + e], s_odd, 0, 0, 0);
        else
          s = __builtin_amdgcn_mfma_f32_32x32x2f32(k[e], q[4 * j + e], s, 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    s += s_odd;
    // the values have arrived by now; settled before the next keys go out, so that the compiler's
    // waits for them never count those
#pragma unroll
    for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(v[r]));
    __builtin_amdgcn_s_waitcnt(0xC07F);  // every LDS read of this block is done (lgkmcnt 0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (t + kWaves < n_blk) {
      locate(j0 + kWaves * kKeys);
      MPIC_WAIT_VMCNT(0);
      stage_keys();
    }
    __builtin_amdgcn_sched_barrier(0);
    if (j0 + kKeys - 1 > lo_pos || j0 + kKeys > key1) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int j = j0 + (r >> 2) * 8 + hi * 4 + (r & 3);
        s[r] = j <= my_pos && j < key1 ? s[r] : -INFINITY;
      }
    }
    float m_blk = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) m_blk = fmaxf(m_blk, s[r]);
    const float m_new = fmaxf(m_run, max_across_halves(m_blk));
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // nothing visible yet: every weight below is exp2(-inf)
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
      const float alpha = weight(m_run - m_ref);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < G::kBlocks; ++db) acc_o[db] *= alpha;
      m_run = m_new;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = weight(s[r] - m_ref);
      if (r % 4 == 3) l_run += (s[r - 3] + s[r - 2]) + (s[r - 1] + s[r]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int db = 0; db < G::kBlocks; ++db) acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[r][db], s[r], acc_o[db], 0, 0, 0);
  }

  // A key that a query does not see has weight 0, and 0 times an infinity or NaN of its value row is no
  // number.  A wavefront whose result is not finite takes its keys once more, without the matrix
  // cores, and adds each value row to the queries that see it.  (As a second pass of the loop above the
  // registers spilled: one image 56.9 -> 62.2 us.)
  float finite = 0.f;
#pragma unroll
  for (int db = 0; db < G::kBlocks; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) finite = fmaf(acc_o[db][r], 0.f, finite);
  if (__builtin_amdgcn_ballot_w64(!(finite == 0.f)) != 0) {
    const float m_ref = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
    for (int db = 0; db < G::kBlocks; ++db) acc_o[db] = f32x16{0};
    for (int j = key0 + wave * kKeys; j < key1; j += (j - key0) % kKeys == kKeys - 1 ? (kWaves - 1) * kKeys + 1 : 1) {
      if ((j - key0) % kKeys == 0) locate(j);
      const int key = (j - key0) % kKeys;
      const f32x4* k = reinterpret_cast<const f32x4*>(from_lane(kp, key)) + hi;
      const int of = kLazy ? __shfl(inst, key) : -1;
      const float* ct = kLazy && of >= 0 ? src.rope_cos + static_cast<int64_t>(of) * (D / 2) : nullptr;
      const float* st = kLazy && of >= 0 ? src.rope_sin + static_cast<int64_t>(of) * (D / 2) : nullptr;
      float dot = 0.f;
#pragma unroll
      for (int i = 0; i < D / 16; ++i) {  // chunk 2 i + hi and its partner half a row further
        f32x4 x = k[2 * i], y = k[2 * i + G::kChunks / 2];
        if (kLazy && of >= 0) {
          const int ch = 2 * i + hi;
          if (src.interleaved) {
            auto turn = [&](f32x4 u, int c2) {
              const float c0 = ct[2 * c2], s0 = st[2 * c2], c1 = ct[2 * c2 + 1], s1 = st[2 * c2 + 1];
              return f32x4{u[0] * c0 - u[1] * s0, u[0] * s0 + u[1] * c0, u[2] * c1 - u[3] * s1, u[2] * s1 + u[3] * c1};
            };
            x = turn(x, ch);
            y = turn(y, ch + G::kChunks / 2);
          } else {
            const f32x4 cc = *reinterpret_cast<const f32x4*>(ct + 4 * ch), ss = *reinterpret_cast<const f32x4*>(st + 4 * ch);
            const f32x4 u = x;
            x = u * cc - y * ss;
            y = u * ss + y * cc;
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) dot = fmaf(q[4 * i + e], x[e], fmaf(q[4 * (i + D / 16) + e], y[e], dot));
        __builtin_amdgcn_sched_barrier(0);
      }
      const float w = weight(dot + __shfl_xor(dot, 32) - m_ref);
      const char* v = from_lane(vp, key);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const vrow x = *reinterpret_cast<const vrow*>(v + ((r >> 2) * 8 + here(hi) * 4 + (r & 3)) * (G::kBlocks * 4));
#pragma unroll
        for (int db = 0; db < G::kBlocks; ++db) acc_o[db][r] = j <= my_pos ? fmaf(w, x[db], acc_o[db][r]) : acc_o[db][r];
        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- merge the wavefronts: partial results as [wave][coordinate][column] ----
  const float l_wave = sum_across_halves(l_run);
  __syncthreads();
  float* part = reinterpret_cast<float*>(lds);
  float* m_of = part + kWaves * D * kCols;
  float* l_of = m_of + kWaves * kCols;
#pragma unroll
  for (int db = 0; db < G::kBlocks; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = (r >> 2) * 8 + hi * 4 + (r & 3);
      part[(wave * D + G::kBlocks * i + db) * kCols + col] = acc_o[db][r];
    }
  if (hi == 0) {
    m_of[wave * kCols + col] = m_run;
    l_of[wave * kCols + col] = l_wave;
  }
  __syncthreads();
  const int mc = tid & 31, d0 = (tid >> 5) * G::kPerThread;
  float m_tot = -INFINITY;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) m_tot = fmaxf(m_tot, m_of[w * kCols + mc]);
  float l_tot = 0.f;
  float o[G::kPerThread];
#pragma unroll
  for (int i = 0; i < G::kPerThread; ++i) o[i] = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float mw = m_of[w * kCols + mc];
    const float wgt = mw == -INFINITY ? 0.f : weight(mw - m_tot);
    l_tot = fmaf(wgt, l_of[w * kCols + mc], l_tot);
#pragma unroll
    for (int i = 0; i < G::kPerThread; ++i) o[i] = fmaf(wgt, part[(w * D + d0 + i) * kCols + mc], o[i]);
  }
  emit(mc, d0, o, m_tot, l_tot);
}

}  // namespace f32tile
}  // namespace mpic
