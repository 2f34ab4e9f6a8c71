// Decode-step attention of libmpic over a linked context (gfx950).
//
// App. A (autoregressive generation): after the prefill the model emits one token at a
// time; the query of the new token attends to every cached position and, its key and
// value being appended to the cache, to itself.  Here the cache is the context that the
// linker wrote (Fig. 7 step 2), contiguous or paged, and the new token of request b sits
// at position N_b.
//
// The step reads every context row once and does 4*D flops per (query head, key), so it
// is bound by HBM bandwidth.  Work decomposition of the bf16 kernel: the keys of one
// (request, kv head) are cut into splits; a workgroup of four wavefronts owns one split
// and its wavefronts take the 32-key blocks of the split in turn, each through its own
// double-buffered LDS staging area filled by direct global->LDS loads (no barrier inside
// the loop: a wavefront only reads what it loaded itself).  The query heads of the kv
// group are the columns of a 32-column matrix-core tile (S^T = K.Q^T, O^T = V^T.P^T, the
// transposed formulation of the prefill kernel: softmax statistics are per-lane
// scalars).  The four wavefronts merge their partial results through LDS.  Where the keys are
// not split, the workgroup adds the new token itself and writes the output; otherwise it writes one
// (O, log-sum-exp) partial per split, and a second small kernel merges the splits and adds the new
// token.  (Merging in the workgroup that arrives last, with partial results that go past the L2s and a
// counter, takes longer than that launch: 14.2 us against 13.5 for 2.6K tokens with 32 kv heads, 36.5
// against 33.1 for the 18K-token batch of 4.)
#include <type_traits>

#include "common.h"
#include "f32_tile.h"
#include "wave_ops.h"

namespace mpic {
namespace {

constexpr int D = 128;
constexpr int WAVES = 4;
constexpr int THREADS = WAVES * 64;
constexpr int BN = 32;                           // keys per wavefront block
constexpr int ROW_BYTES = D * 2;
constexpr int TILE_BYTES = BN * ROW_BYTES;       // one staged K (or V) block: 8 KB
constexpr int STAGE_BYTES = 2 * TILE_BYTES;      // K block followed by V block
constexpr int STAGES = 2;                        // blocks in flight per wavefront: STAGES - 1
constexpr int WAVE_LDS = STAGES * STAGE_BYTES;
constexpr int LDS_BYTES = WAVES * WAVE_LDS;
constexpr int LOADS_PER_BLOCK = 16;              // direct loads per wavefront and block
constexpr int FINISH_AT = WAVES * 32 * D + 2 * WAVES * 32;  // LDS of the rows of an unsplit step, in floats: behind the merge area
constexpr float kSlack = 8.0f;                   // lazy-rescale threshold, log2 units
static_assert(kDecodeBlockKeys % BN == 0, "a split is a whole number of key blocks");
static_assert(LDS_BYTES <= 160 * 1024 && LOADS_PER_BLOCK * (STAGES - 1) <= 63, "LDS size / load counter range");
static_assert((FINISH_AT + 32 * D + 32) * 4 <= LDS_BYTES, "merge area and finished rows must fit the staging area");

// wait until at most `blocks` blocks of loads are outstanding; the empty asm keeps the
// compiler from moving an LDS read above the wait
__device__ inline void wait_loads(int blocks) {
  if (blocks >= 3) {
    MPIC_WAIT_VMCNT(48);
  } else if (blocks == 2) {
    MPIC_WAIT_VMCNT(32);
  } else if (blocks == 1) {
    MPIC_WAIT_VMCNT(16);
  } else {
    MPIC_WAIT_VMCNT(0);
  }
  asm volatile("" ::: "memory");
}
static_assert(LOADS_PER_BLOCK == 16, "wait_loads spells the count out");

// The end of an unsplit step: the context's share of output rows h0 .. h0 + n_cols - 1 of request b
// (normalised, [n_cols][kD], and its log-sum-exp, both in LDS; any_key = false: the request has no
// context) and the new token's own term give the rows.  Called by the whole workgroup, once its LDS
// writes are visible.  Saves the merge launch, 2.3 us (28 heads over 4, 64 keys 8.0 -> 6.1 us; fp32 with 4
// heads, 250 keys 12.5 -> 10.4).
template <typename T, int kD, int kThreads>
__device__ inline void finish_rows(const DecodeArgs& a, int b, int g, int h0, int n_cols, bool any_key, const float* part_o,
                                   const float* part_lse) {
  constexpr int kLanes = kD / 4;  // threads per output row
  typedef T t4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, d0 = tid % kLanes * 4;
  const int64_t kv = (static_cast<int64_t>(b) * a.n_kv_heads + g) * kD + d0;
  f32x4 k = f32x4{0}, v = f32x4{0};
  if (a.new_k) {
    k = __builtin_convertvector(*reinterpret_cast<const t4*>(static_cast<const T*>(a.new_k) + kv), f32x4);
    v = __builtin_convertvector(*reinterpret_cast<const t4*>(static_cast<const T*>(a.new_v) + kv), f32x4);
  }
  for (int c = tid / kLanes; c < n_cols; c += kThreads / kLanes) {
    const int64_t row = static_cast<int64_t>(b) * a.n_q_heads + h0 + c;
    float self = -INFINITY;
    if (a.new_k) {
      const f32x4 q = __builtin_convertvector(*reinterpret_cast<const t4*>(static_cast<const T*>(a.q) + row * kD + d0), f32x4);
      self = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) self = fmaf(q[e], k[e], self);
#pragma unroll
      for (int off = kLanes / 2; off > 0; off >>= 1) self += __shfl_xor(self, off);
      self *= a.scale;
    }
    const float lse = any_key ? part_lse[c] : -INFINITY;
    const float m = any_key ? fmaxf(lse, self) : self;  // (a maximum would drop a self that is no number)
    f32x4 o = f32x4{0};
    float z = 0.f;
    if (m != -INFINITY) {
      if (any_key) {
        z = expf(lse - m);
        o = *reinterpret_cast<const f32x4*>(part_o + c * kD + d0) * z;
      }
      if (a.new_k) {
        const float w = expf(self - m);
        z += w;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = fmaf(w, v[e], o[e]);
      }
      o /= z;
    }
    *reinterpret_cast<t4*>(static_cast<T*>(a.out) + row * kD + d0) = __builtin_convertvector(o, t4);
    if (a.lse && d0 == 0) a.lse[row] = m == -INFINITY ? -INFINITY : m + logf(z);
  }
}

// Extra = LazyRefs (lazy_rope contexts): the wavefronts walk the request's 32-key blocks of the
// plan (KeyBlock: one source and one missing shift per block, slots past n_valid are padding),
// stage each block from its source's base address, and turn the query back by the block's shift
// whenever it changes, <Rot(-s) q, k> = <q, Rot(s) k>; a.keys_per_split then counts slots of
// those blocks.
struct NoLazy {};
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// kUnsplit: a.n_splits is 1 and the kernel writes the output rows (a kernel of its own, since the longer code
// costs the split steps 0.3 us).
template <typename Extra, bool kUnsplit>
__global__ __launch_bounds__(THREADS) void decode_bf16_kernel(DecodeArgs a, Extra extra) {
  constexpr bool kLazy = std::is_same<Extra, LazyRefs>::value;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int col = lane & 31;
  const int hi = lane >> 5;
  const int group = a.n_q_heads / a.n_kv_heads;
  const int col_blocks = (group + 31) / 32;
  const int split = blockIdx.x;
  const int g = blockIdx.y / col_blocks;
  const int cb = blockIdx.y % col_blocks;
  const int b = blockIdx.z;
  // keys of this request, or (lazy) slots of its key blocks
  int n_ctx = a.ctx_off[b + 1] - a.ctx_off[b];
  int vb0 = 0;
  if constexpr (kLazy) {
    n_ctx = (extra.first[b + 1] - extra.first[b]) * BN;
    vb0 = extra.first[b] + split * (a.keys_per_split / BN);
  }
  const int key0 = split * a.keys_per_split;
  const int n_cols = min(32, group - cb * 32);
  float* const fin = reinterpret_cast<float*>(lds) + FINISH_AT;
  if (key0 >= n_ctx) {  // this request has fewer splits (the whole workgroup leaves), or no context
    if constexpr (kUnsplit) finish_rows<__bf16, D, THREADS>(a, b, g, g * group + cb * 32, n_cols, false, fin, fin);
    return;
  }
  const int n_keys = min(n_ctx, key0 + a.keys_per_split) - key0;
  const int n_blk = (n_keys + BN - 1) / BN;

  const __attribute__((address_space(4))) uint32_t* off_of;
  if constexpr (kLazy) {
    off_of = (const __attribute__((address_space(4))) uint32_t*)(extra.voff + static_cast<int64_t>(vb0) * BN);
  } else {
    off_of = (const __attribute__((address_space(4))) uint32_t*)(a.kv_off16 + a.ctx_off[b] + key0);
  }
  auto desc_of = [&](int blk) __attribute__((always_inline)) {
    blk = blk < n_blk ? blk : n_blk - 1;
    KeyBlock d{};
    if constexpr (kLazy) {
      const i32x4 raw = *(const __attribute__((address_space(4))) i32x4*)(extra.blocks + vb0 + blk);
      d.pos0 = raw[0];
      d.n_valid = raw[1];
      d.inst = raw[2];
    }
    return d;
  };
  const char* kbase_ctx = static_cast<const char*>(a.k_ctx) + g * ROW_BYTES;
  const char* vbase_ctx = static_cast<const char*>(a.v_ctx) + g * ROW_BYTES;
  char* my_lds = lds + wave * WAVE_LDS;
  const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(MPIC_LDS_PTR(char, my_lds)));

  // ---- this lane's query column: head cb*32 + col of the kv group (columns past the group
  // repeat its first head and are never written) ----
  const int in_group = cb * 32 + col;
  const bool valid = in_group < group;
  const int head = g * group + (valid ? in_group : cb * 32);
  const __bf16* qp = static_cast<const __bf16*>(a.q) + (static_cast<int64_t>(b) * a.n_q_heads + head) * D;
  bf16x8 qf[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16 + hi * 8);
  // lazy: the query as handed over, and the query turned back by the shift of instance `inst`
  // (fp32 arithmetic, one rounding).  This lane holds coordinates d = 16*ks + 8*hi + e: a
  // rotate-half pair (d, d + 64) is (q[ks], q[ks + 4]), an interleaved pair two neighbours.
  bf16x8 q0[8];
  int q_inst = -1;
  if constexpr (kLazy) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) q0[ks] = qf[ks];
  }
  auto turn_back = [&](int inst) __attribute__((always_inline)) {
    if (inst < 0) {
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) qf[ks] = q0[ks];
      return;
    }
    const float* cb = nullptr;
    const float* sb = nullptr;
    if constexpr (kLazy) {
      cb = extra.rope_cos + static_cast<int64_t>(inst) * (D / 2);
      sb = extra.rope_sin + static_cast<int64_t>(inst) * (D / 2);
    }
    if (a.interleaved) {
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const f32x4 c = *reinterpret_cast<const f32x4*>(cb + ks * 8 + hi * 4);
        const f32x4 s = *reinterpret_cast<const f32x4*>(sb + ks * 8 + hi * 4);
        const f32x8 x = __builtin_convertvector(q0[ks], f32x8);
        f32x8 y;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          y[2 * i] = x[2 * i] * c[i] + x[2 * i + 1] * s[i];
          y[2 * i + 1] = x[2 * i + 1] * c[i] - x[2 * i] * s[i];
        }
        qf[ks] = __builtin_convertvector(y, bf16x8);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const f32x8 c = *reinterpret_cast<const f32x8*>(cb + ks * 16 + hi * 8);
        const f32x8 s = *reinterpret_cast<const f32x8*>(sb + ks * 16 + hi * 8);
        const f32x8 x0 = __builtin_convertvector(q0[ks], f32x8);
        const f32x8 x1 = __builtin_convertvector(q0[ks + 4], f32x8);
        qf[ks] = __builtin_convertvector(x0 * c + x1 * s, bf16x8);
        qf[ks + 4] = __builtin_convertvector(x1 * c - x0 * s, bf16x8);
      }
    }
  };

  const float scale_log2 = a.scale * 1.4426950408889634f;
  float m_run = -INFINITY;
  float l_run = 0.f;
  f32x16 acc_o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc_o[i] = f32x16{0};

  // ---- loader: load p (0..7) stages rows 4p..4p+3 of K and of V; lane i owns LDS column
  // i&15 of row 4p + (i>>4).  Logical column c of row r is stored at column c ^ swizzle(r):
  // K swizzle = r & 15, V swizzle = (r & 3) << 2 (conflict-free fragment reads below) ----
  const int ld_sub = lane >> 4;
  const uint32_t ld_col = lane & 15;
  const uint32_t ld_k16 = ld_col ^ ld_sub;        // ^ ((p & 3) << 2)
  const uint32_t ld_v16 = ld_col ^ (ld_sub << 2);
  struct Rows {
    u32x8_a4 r[4];
    const char* kb;  // lazy: base of the block's rows (context, or the chunk's cache)
    const char* vb;
  };
  auto fetch_rows = [&](int blk) {
    blk = blk < n_blk ? blk : n_blk - 1;
    Rows x;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      x.r[i] = *reinterpret_cast<const __attribute__((address_space(4))) u32x8_a4*>(off_of + blk * BN + i * 8);
    if constexpr (kLazy) {
      const int inst = desc_of(blk).inst;
      const bool in_ctx = inst < 0 || !extra.by_ref;
      x.kb = (in_ctx ? static_cast<const char*>(a.k_ctx) : static_cast<const char*>(extra.k[inst])) + g * ROW_BYTES;
      x.vb = (in_ctx ? static_cast<const char*>(a.v_ctx) : static_cast<const char*>(extra.v[inst])) + g * ROW_BYTES;
    }
    return x;
  };
  auto issue_loads = [&](const Rows& cur, int stage) {
    const char* kbase = kbase_ctx;
    const char* vbase = vbase_ctx;
    if constexpr (kLazy) {
      kbase = cur.kb;
      vbase = cur.vb;
    }
    const uint32_t dst = lds_base + stage * STAGE_BYTES;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const u32x8_a4 q8 = cur.r[p >> 1];
      const int o = (p & 1) * 4;
      const uint32_t r16 = ld_sub == 0 ? q8[o] : ld_sub == 1 ? q8[o + 1] : ld_sub == 2 ? q8[o + 2] : q8[o + 3];
      load_to_lds_16B_nt(kbase + (static_cast<uint64_t>(r16 + (ld_k16 ^ ((p & 3) << 2))) << 4), dst + p * 4 * ROW_BYTES);
      load_to_lds_16B_nt(vbase + (static_cast<uint64_t>(r16 + ld_v16) << 4), dst + TILE_BYTES + p * 4 * ROW_BYTES);
    }
  };

  // ---- LDS byte offsets of this lane's operand fragments (layout of
  // v_mfma_f32_32x32x16_bf16: A[i][k] lane i + 32*(k/8), element k%8; B likewise with the
  // column in place of i; C[i][j] lane j + 32*((i/4)%2), register (i/8)*4 + i%4) ----
  const int k_row_off = col * ROW_BYTES;
  const int k_col_x = hi ^ (col & 15);
  const int i16 = lane & 15;
  const int v_row = hi * 4 + (i16 >> 2);
  const int v_col_x = ((((lane >> 4) & 1) << 1) | ((i16 & 3) >> 1)) ^ ((v_row & 3) << 2);
  const int v_off = TILE_BYTES + v_row * ROW_BYTES + (i16 & 1) * 8;

  // every ordinary load is complete before the first direct load: from here on the
  // outstanding-load counter only counts staging traffic
  MPIC_WAIT_VMCNT(0);
  __builtin_amdgcn_sched_barrier(0);

  // Software pipeline: the loads of the next STAGES-1 blocks of this wavefront are in
  // flight while one block is consumed; row offsets (scalar loads) are fetched one block
  // ahead of the loads that use them.
  const int first = wave;
  const int my_blocks = first < n_blk ? (n_blk - first + WAVES - 1) / WAVES : 0;
  Rows rows = fetch_rows(first);
  int issued = 0;
#pragma unroll
  for (int i = 0; i < STAGES - 1; ++i)
    if (issued < my_blocks) {
      issue_loads(rows, issued % STAGES);
      ++issued;
      rows = fetch_rows(first + issued * WAVES);
    }
  for (int it = 0; it < my_blocks; ++it) {
    const int blk = first + it * WAVES;
    const int stage = it % STAGES;
    if (issued < my_blocks) {
      issue_loads(rows, issued % STAGES);
      ++issued;
      rows = fetch_rows(first + issued * WAVES);
    }
    wait_loads(issued - it - 1);
    const char* st = my_lds + stage * STAGE_BYTES;
    KeyBlock kd{};
    if constexpr (kLazy) {
      kd = desc_of(blk);
      if (kd.inst != q_inst) {  // the keys of this block lack another shift than the last block's
        turn_back(kd.inst);
        q_inst = kd.inst;
      }
    }

    // S^T = K . Q^T for 32 keys x 32 query columns
    f32x16 acc_s = f32x16{0};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const bf16x8 kf = *reinterpret_cast<const bf16x8*>(st + k_row_off + ((k_col_x ^ (ks << 1)) << 4));
      acc_s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], acc_s, 0, 0, 0);
    }
    // keys past the end of the context (ragged last block) take no weight
    if constexpr (kLazy) {
      if (kd.n_valid < BN) {  // slots past the block's keys are padding
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int slot = (v >> 2) * 8 + hi * 4 + (v & 3);
          acc_s[v] = slot < kd.n_valid ? acc_s[v] : -INFINITY;
        }
      }
    } else {
    const int j0 = blk * BN;
    if (j0 + BN > n_keys) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = j0 + (v >> 2) * 8 + hi * 4 + (v & 3);
        acc_s[v] = key < n_keys ? acc_s[v] : -INFINITY;
      }
    }
    }
    float m_blk = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) m_blk = fmaxf(m_blk, acc_s[v]);
    m_blk = max_across_halves(m_blk);
    // lazy rescale: the reference maximum only moves when a block maximum exceeds it by
    // more than kSlack (log2 units); exact because numerator and denominator share it
    if (__builtin_amdgcn_ballot_w64((m_blk - m_run) * scale_log2 > kSlack) != 0) {
      const float m_new = fmaxf(m_run, m_blk);
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db) acc_o[db] *= alpha;
    }
    const float m_scaled = m_run * scale_log2;
    bf16x8 pf[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f32x8 p;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = __builtin_amdgcn_exp2f(fmaf(acc_s[half * 8 + e], scale_log2, -m_scaled));
        l_run += p[e];
      }
      pf[half] = __builtin_convertvector(p, bf16x8);
    }
    // O^T += V^T . P^T, 16 keys per step; V^T fragments through the LDS transpose read
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const char* vp = st + v_off + kh * 16 * ROW_BYTES + ((v_col_x ^ (db << 2)) << 4);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(MPIC_LDS_PTR(s16x4, vp));
        const s16x4 up = __builtin_amdgcn_ds_read_tr16_b64_v4i16(MPIC_LDS_PTR(s16x4, vp + 8 * ROW_BYTES));
        const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7));
        acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[kh], acc_o[db], 0, 0, 0);
      }
  }

  // ---- merge the four wavefronts through LDS (the staging areas are free now) ----
  const float l_wave = sum_across_halves(l_run);
  __syncthreads();
  float* m_o = reinterpret_cast<float*>(lds);               // [WAVES][32 columns][D]
  float* m_m = m_o + WAVES * 32 * D;                        // [WAVES][32]
  float* m_l = m_m + WAVES * 32;                            // [WAVES][32]
  if (valid) {  // (rows of 512 bytes conflict in the LDS banks: only the columns that are merged below)
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc_o[db][q4 * 4 + e];
        *reinterpret_cast<f32x4*>(m_o + (wave * 32 + col) * D + db * 32 + q4 * 8 + hi * 4) = o;
      }
  }
  if (hi == 0) {
    m_m[wave * 32 + col] = m_run;
    m_l[wave * 32 + col] = l_wave;
  }
  __syncthreads();
  {
    const int d0 = (tid & 7) * 16;  // this thread's 16 output coordinates
    for (int c = tid >> 3; c < 32; c += THREADS / 8) {  // of these columns
      const int hg = cb * 32 + c;
      if (hg >= group) break;
      float m_tot = -INFINITY;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) m_tot = fmaxf(m_tot, m_m[w * 32 + c]);
      float wgt[WAVES];
      float l_tot = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const float mw = m_m[w * 32 + c];
        wgt[w] = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mw - m_tot) * scale_log2);
        l_tot += wgt[w] * m_l[w * 32 + c];
      }
      const float inv = 1.f / l_tot;  // a split holds at least one key, so l_tot > 0
      const int64_t part = (static_cast<int64_t>(b) * a.n_q_heads + g * group + hg) * a.n_splits + split;
      const float lse = m_tot * a.scale + logf(l_tot);
#pragma unroll
      for (int i = 0; i < 16; i += 4) {
        f32x4 acc = f32x4{0};
#pragma unroll
        for (int w = 0; w < WAVES; ++w) acc += wgt[w] * *reinterpret_cast<const f32x4*>(m_o + (w * 32 + c) * D + d0 + i);
        if constexpr (kUnsplit) {
          *reinterpret_cast<f32x4*>(fin + c * D + d0 + i) = acc * inv;
        } else {
          *reinterpret_cast<f32x4*>(a.ws_o + part * D + d0 + i) = acc * inv;
        }
      }
      if ((tid & 7) == 0) {
        if constexpr (kUnsplit) {
          fin[32 * D + c] = lse;
        } else {
          a.ws_lse[part] = lse;
        }
      }
    }
  }
  if constexpr (kUnsplit) {
    __syncthreads();
    finish_rows<__bf16, D, THREADS>(a, b, g, g * group + cb * 32, n_cols, true, fin, fin + 32 * D);
  }
}

// Merge the splits of one (request, query head) and the new token itself; one thread per
// output coordinate.  The partials were written by other compute units, so every read
// here goes to memory: the split weights are computed once by the first wavefront (one
// split per lane) and the partial outputs are fetched eight at a time before they are
// used, so that the latencies overlap instead of adding up.
template <typename T, int kD>
__global__ __launch_bounds__(kD) void decode_merge_kernel(DecodeArgs a) {
  constexpr int kMaxSplits = 1024;
  __shared__ float red[kD / 64];
  __shared__ float wgt[kMaxSplits];
  __shared__ float stat[2];  // reference maximum, denominator
  const int d = threadIdx.x;
  const int64_t row = blockIdx.x;  // b * Hq + h
  const int b = static_cast<int>(row / a.n_q_heads);
  const int h = static_cast<int>(row % a.n_q_heads);
  const int g = h / (a.n_q_heads / a.n_kv_heads);
  // keys of the request, or (lazy_rope, bf16) slots of its 32-key blocks
  const int n_ctx = a.blk_first ? (a.blk_first[b + 1] - a.blk_first[b]) * 32 : a.ctx_off[b + 1] - a.ctx_off[b];
  const int n_s = (n_ctx + a.keys_per_split - 1) / a.keys_per_split;
  // The first log-sum-exps and partial outputs are fetched right here, before the weights are known and
  // whether or not the request has that many splits (the others are not used): they and the tables
  // arrive together instead of one after the other (with the narrower LDS merge of the main kernel
  // 16.6 -> 13.6 us for a step over 2.6K tokens with 32 kv heads).
  constexpr int kAhead = 8;
  const float* po = a.ws_o + row * a.n_splits * kD + d;
  const float lse0 = a.ws_lse[row * a.n_splits + min(d, a.n_splits - 1)];
  float x0[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) x0[i] = po[static_cast<int64_t>(min(i, a.n_splits - 1)) * kD];
  float self = -INFINITY;
  float v_new = 0.f;
  if (a.new_k) {
    const int64_t kv = (static_cast<int64_t>(b) * a.n_kv_heads + g) * kD + d;
    float part = static_cast<float>(static_cast<const T*>(a.q)[row * kD + d]) *
                 static_cast<float>(static_cast<const T*>(a.new_k)[kv]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
    if ((d & 63) == 0) red[d >> 6] = part;
    v_new = static_cast<float>(static_cast<const T*>(a.new_v)[kv]);
  }
  __syncthreads();
  if (a.new_k) {
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < kD / 64; ++i) dot += red[i];
    self = dot * a.scale;
  }
  if (d < 64) {
    // lane l owns splits l, l + 64, ...
    float m = d < n_s ? fmaxf(self, lse0) : self;
    for (int s = d + 64; s < n_s; s += 64) m = fmaxf(m, a.ws_lse[row * a.n_splits + s]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    float z = 0.f;
    if (m != -INFINITY) {
      if (d < n_s) {
        z = expf(lse0 - m);
        wgt[d] = z;
      }
      for (int s = d + 64; s < n_s; s += 64) {
        const float w = expf(a.ws_lse[row * a.n_splits + s] - m);
        wgt[s] = w;
        z += w;
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) z += __shfl_xor(z, off);
    if (d == 0) {
      stat[0] = m;
      stat[1] = z;
    }
  }
  __syncthreads();
  const float m = stat[0];
  float z = stat[1];
  float o = 0.f;
  if (m != -INFINITY) {
    int s = min(n_s, kAhead);
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (i < s) o = fmaf(wgt[i], x0[i], o);
    for (; s + 8 <= n_s; s += 8) {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = po[static_cast<int64_t>(s + i) * kD];
#pragma unroll
      for (int i = 0; i < 8; ++i) o = fmaf(wgt[s + i], x[i], o);
    }
    for (; s < n_s; ++s) o = fmaf(wgt[s], po[static_cast<int64_t>(s) * kD], o);
    if (a.new_k) {
      const float w = expf(self - m);
      z += w;
      o = fmaf(w, v_new, o);
    }
    o /= z;
  }
  static_cast<T*>(a.out)[row * kD + d] = static_cast<T>(o);
  if (a.lse && d == 0) a.lse[row] = m == -INFINITY ? -INFINITY : m + logf(z);
}

// fp32 path: the query heads of a kv group are the columns of one fp32 tile (f32_tile.h), a
// workgroup owns one split of the keys.  kLazy (lazy_rope contexts): stored keys are turned to
// their position as they are read, in fp32; refs.by_ref: stored rows are read in their caches.
template <int kD, bool kLazy, bool kUnsplit>
__global__ __launch_bounds__(f32tile::kThreads, 2) void decode_f32_kernel(DecodeArgs a, LazyRefs refs) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int group = a.n_q_heads / a.n_kv_heads;
  const int col_blocks = (group + f32tile::kCols - 1) / f32tile::kCols;
  const int split = blockIdx.x % a.n_splits;
  const int g = blockIdx.y / col_blocks;
  const int h0 = g * group + blockIdx.y % col_blocks * f32tile::kCols;
  const int n_cols = min(f32tile::kCols, (g + 1) * group - h0);
  const int b = blockIdx.x / a.n_splits;
  const int n_ctx = a.ctx_off[b + 1] - a.ctx_off[b];
  const int key0 = split * a.keys_per_split;
  float* const fin = reinterpret_cast<float*>(lds);
  if (key0 >= n_ctx) {  // this request has fewer splits, or no context
    if constexpr (kUnsplit) finish_rows<float, kD, f32tile::kThreads>(a, b, g, h0, n_cols, false, fin, fin);
    return;
  }
  const int key1 = min(n_ctx, key0 + a.keys_per_split);
  const int64_t row0 = static_cast<int64_t>(b) * a.n_q_heads + h0;
  f32tile::Rows src{};
  src.off16 = a.kv_off16 + a.ctx_off[b];
  src.k = static_cast<const char*>(a.k_ctx) + static_cast<int64_t>(g) * kD * 4;
  src.v = static_cast<const char*>(a.v_ctx) + static_cast<int64_t>(g) * kD * 4;
  if constexpr (kLazy) {
    src.inst = a.src_inst + a.ctx_off[b];
    src.row = a.src_row + a.ctx_off[b];
    src.rope_cos = a.rope_cos;
    src.rope_sin = a.rope_sin;
    src.refs = &refs;
    src.head_bytes = static_cast<int64_t>(g) * kD * 4;
    src.row_bytes = static_cast<int64_t>(a.n_kv_heads) * kD * 4;
    src.interleaved = a.interleaved;
  }
  f32tile::attend<kD, kLazy, kD == 128>(src, [&](int c) { return static_cast<const char*>(a.q) + (row0 + min(c, n_cols - 1)) * (kD * 4); },
                                        [](float(&)[kD / 2]) {}, key1 - 1, key0, key1, a.scale, lds,
                                        [&](int c, int d0, const float(&o)[f32tile::Geo<kD>::kPerThread], float m, float l) {
    if constexpr (kUnsplit) __syncthreads();  // (every thread is here once: what lies in LDS has been read)
    if (c >= n_cols) return;
    const int64_t part = (row0 + c) * a.n_splits + split;
    const float inv = 1.f / l;
#pragma unroll
    for (int i = 0; i < f32tile::Geo<kD>::kPerThread; i += 4) {
      const f32x4 x = f32x4{o[i], o[i + 1], o[i + 2], o[i + 3]} * inv;
      if constexpr (kUnsplit) {
        *reinterpret_cast<f32x4*>(fin + c * kD + d0 + i) = x;
      } else {
        *reinterpret_cast<f32x4*>(a.ws_o + part * kD + d0 + i) = x;
      }
    }
    if (d0 != 0) return;
    const float lse = m * a.scale + logf(l);
    if constexpr (kUnsplit) {
      fin[f32tile::kCols * kD + c] = lse;
    } else {
      a.ws_lse[part] = lse;
    }
  });
  if constexpr (kUnsplit) {
    __syncthreads();
    finish_rows<float, kD, f32tile::kThreads>(a, b, g, h0, n_cols, true, fin, fin + f32tile::kCols * kD);
  }
}

template <int kD, bool kLazy, bool kUnsplit>
hipError_t launch_f32_kernel(const DecodeArgs& a, const LazyRefs& refs, int dev, hipStream_t stream) {
  constexpr int kLds = f32tile::Geo<kD>::kLdsBytes;
  static LdsOptIn opt_in;
  const hipError_t e = opt_in.ensure(dev, [] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(decode_f32_kernel<kD, kLazy, kUnsplit>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  });
  if (e != hipSuccess) return e;
  const int group = a.n_q_heads / a.n_kv_heads;
  const dim3 grid(static_cast<unsigned>(a.n_splits) * a.n_requests, a.n_kv_heads * ((group + f32tile::kCols - 1) / f32tile::kCols));
  hipLaunchKernelGGL((decode_f32_kernel<kD, kLazy, kUnsplit>), grid, dim3(f32tile::kThreads), kLds, stream, a, refs);
  return hipSuccess;
}

template <int kD, bool kLazy>
hipError_t launch_f32(const DecodeArgs& a, const LazyRefs& refs, int dev, hipStream_t stream) {
  const hipError_t e = a.n_splits == 1 ? launch_f32_kernel<kD, kLazy, true>(a, refs, dev, stream)
                                       : launch_f32_kernel<kD, kLazy, false>(a, refs, dev, stream);
  if (e != hipSuccess) return e;
  if (a.n_splits > 1)
    hipLaunchKernelGGL((decode_merge_kernel<float, kD>), dim3(static_cast<unsigned>(a.n_requests) * a.n_q_heads), dim3(kD), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

// Scratch of mpic_decode_attn_static: partial results of the key splits for callers that must
// not allocate.  The array exists once per GPU for the life of the process.  In host code its
// name is only a handle: the device address comes from hipGetSymbolAddress, looked up once per
// device with that device current, and only that address is handed to kernels.
constexpr size_t kStaticScratchBytes = size_t{8} << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t decode_static_scratch(float** ptr, size_t* bytes) {
  static std::mutex mu;
  static void* addr[64] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = static_cast<float*>(addr[dev]);
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

hipError_t launch_decode(int dtype, const DecodeArgs& a, const LazyRefs* lazy, hipStream_t stream) {
  const int64_t rows = static_cast<int64_t>(a.n_requests) * a.n_q_heads;
  if (rows <= 0) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dtype == MPIC_F32) {
    if (a.head_dim == 64)
      return lazy ? launch_f32<64, true>(a, *lazy, dev, stream) : launch_f32<64, false>(a, LazyRefs{}, dev, stream);
    return lazy ? launch_f32<128, true>(a, *lazy, dev, stream) : launch_f32<128, false>(a, LazyRefs{}, dev, stream);
  }
  static LdsOptIn opt_in;
  e = opt_in.ensure(dev, [] {
    for (const void* kernel : {reinterpret_cast<const void*>(decode_bf16_kernel<NoLazy, false>), reinterpret_cast<const void*>(decode_bf16_kernel<NoLazy, true>),
                               reinterpret_cast<const void*>(decode_bf16_kernel<LazyRefs, false>), reinterpret_cast<const void*>(decode_bf16_kernel<LazyRefs, true>)}) {
      const hipError_t e0 = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
      if (e0 != hipSuccess) return e0;
    }
    return hipSuccess;
  });
  if (e != hipSuccess) return e;
  const int group = a.n_q_heads / a.n_kv_heads;
  const dim3 grid(a.n_splits, a.n_kv_heads * ((group + 31) / 32), a.n_requests);
  if (lazy) {
    if (a.n_splits == 1)
      hipLaunchKernelGGL((decode_bf16_kernel<LazyRefs, true>), grid, dim3(THREADS), LDS_BYTES, stream, a, *lazy);
    else
      hipLaunchKernelGGL((decode_bf16_kernel<LazyRefs, false>), grid, dim3(THREADS), LDS_BYTES, stream, a, *lazy);
  } else {
    if (a.n_splits == 1)
      hipLaunchKernelGGL((decode_bf16_kernel<NoLazy, true>), grid, dim3(THREADS), LDS_BYTES, stream, a, NoLazy{});
    else
      hipLaunchKernelGGL((decode_bf16_kernel<NoLazy, false>), grid, dim3(THREADS), LDS_BYTES, stream, a, NoLazy{});
  }
  if (a.n_splits > 1)
    hipLaunchKernelGGL((decode_merge_kernel<__bf16, 128>), dim3(static_cast<unsigned>(rows)), dim3(128), 0, stream, a);
  return hipGetLastError();
}

}  // namespace mpic
