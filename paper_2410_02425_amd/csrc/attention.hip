// Attention over the paged KV cache.
//
// Decode: each request row attends to its whole cached context.  The context
// is cut into chunks of DEC_CHUNK positions; one workgroup handles one (row,
// kv head, chunk) and all query heads of that kv head's group, four waves each
// taking one 64-position KV block.  The grid holds only live chunks: work
// item i is the i-th (row, chunk) pair in row-major order, found by a prefix
// sum over the rows' chunk counts.  Partial (max, sum, unnormalised output)
// triples are merged by a combine pass (log-sum-exp rescaling).
//
// Prefill: causal attention of packed prompt rows, one workgroup per 128 query
// rows (fp32, and steps of prompts up to 64 tokens: 64) of one (sequence, head),
// online softmax over 64-key blocks.
#include <type_traits>

#include "device.hpp"

namespace lp {

typedef unsigned int u32x4_tt __attribute__((ext_vector_type(4)));

constexpr int DEC_CHUNK = 256;  // positions per decode workgroup

size_t decode_attention_ws_bytes(int M, int n_heads, int head_dim, int max_ctx) {
  const int splits = (max_ctx + DEC_CHUNK - 1) / DEC_CHUNK;
  return (size_t)M * n_heads * splits * (head_dim + 2) * sizeof(float);
}

int decode_attention_chunks(int ctx) { return (ctx + DEC_CHUNK - 1) / DEC_CHUNK; }

// The fused QKV finish gives each of the 256 threads one q pair of the group
// and requests all its partials at once.
constexpr int DEC_QKV_SPLITS = 6;
bool decode_attention_fuses_qkv(int group, int head_dim, int splits) {
  return group * head_dim / 2 <= 256 && splits >= 1 && splits <= DEC_QKV_SPLITS;
}

// Work item -> (row m, chunk s, slot, context) of a decode workgroup.  Item i
// is the i-th pair in the row-major list of every row's chunks (a row of
// context c has ceil(c / DEC_CHUNK)); contexts are clamped to max_ctx.  Each
// wave computes it on its own: lane l reads row base + l, an inclusive scan
// over the 64 lanes gives the chunks up to that row, and the first lane whose
// running count exceeds the item is the row.  False past the last item.
struct DecodeItem {
  int m, s, slot, ctx, pos;
};
__device__ __forceinline__ bool decode_item(const RowMeta &rows, int M, int max_ctx, int item, DecodeItem &it) {
  const int lane = threadIdx.x & 63;
  int before = 0;
  for (int base = 0; base < M; base += 64) {
    const int r = base + lane;
    const int pos = r < M ? rows.row_pos[r] : 0;
    const int ctx = r < M ? min(pos + 1, max_ctx) : 0;
    const int slot = r < M ? rows.row_slot[r] : 0;
    const int n = ctx > 0 ? (ctx + DEC_CHUNK - 1) / DEC_CHUNK : 0;
    int incl = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    const int total = __shfl(incl, 63, 64);
    const int rel = item - before;
    if (rel < total) {
      const int k = __popcll(__ballot(incl <= rel));  // rows wholly before the item
      it.m = base + k;
      it.s = rel - __shfl(incl - n, k, 64);
      it.slot = __shfl(slot, k, 64);
      it.ctx = __shfl(ctx, k, 64);
      it.pos = __shfl(pos, k, 64);
      return true;
    }
    before += total;
  }
  return false;
}

template <typename T>
struct Vec8;  // 8 consecutive activation elements as fp32
template <>
struct Vec8<bf16_t> {
  static __device__ __forceinline__ void load(const bf16_t *p, float *o) {
    const uint4 u = *(const uint4 *)p;
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
};
template <>
struct Vec8<f16_t> {
  static __device__ __forceinline__ void load(const f16_t *p, float *o) {
    const f16x8_t v = __builtin_bit_cast(f16x8_t, *(const uint4 *)p);
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (float)v[i];
  }
};
template <>
struct Vec8<float> {
  static __device__ __forceinline__ void load(const float *p, float *o) {
    const float4 a = *(const float4 *)p, b = *(const float4 *)(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
  }
};

template <typename T, int HD, int G>
__global__ __launch_bounds__(256) void decode_attn_kernel(const T *__restrict__ q, RowMeta rows,
                                                          KVCache kv, int layer, int M, int n_heads,
                                                          int max_ctx, int max_splits, float *__restrict__ ws) {
  constexpr int DPL = HD / 64;  // dims per lane in P.V
  __shared__ float qs[G][HD];
  __shared__ float ps[4][G][64];
  __shared__ float wm[4][G], wl[4][G];
  __shared__ float wo[4][G][HD];
  // KV head fastest: consecutive block ids, which the dispatcher deals out
  // round-robin over the XCDs, are the heads of one work item
  const int g = blockIdx.x % kv.n_kv_heads;
  DecodeItem it;
  if (!decode_item(rows, M, max_ctx, blockIdx.x / kv.n_kv_heads, it)) return;
  const int m = it.m, s = it.s, slot = it.slot, ctx = it.ctx;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;

  for (int e = threadIdx.x; e < G * HD; e += 256)
    qs[e / HD][e % HD] = Act<T>::ld(q[((int64_t)m * n_heads + g * G) * HD + e]);
  __syncthreads();

  const int blk_pos = s * DEC_CHUNK + wave * 64;  // first position of this wave's block
  const bool active = blk_pos < ctx;
  float mw[G], lw[G], o[G][DPL];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    mw[h] = -INFINITY;
    lw[h] = 0.f;
#pragma unroll
    for (int t = 0; t < DPL; ++t) o[h][t] = 0.f;
  }
  if (active) {
    const int64_t base = kv_block_base(kv, layer, slot, blk_pos, g);
    const T *kb = (const T *)kv.k + base;
    const T *vb = (const T *)kv.v + base;
    const int p = blk_pos + lane;
    const bool valid = p < ctx;
    float sc[G];
#pragma unroll
    for (int h = 0; h < G; ++h) sc[h] = 0.f;
    if (valid) {
#pragma unroll 4
      for (int d = 0; d < HD; d += 8) {
        float kk[8];
        Vec8<T>::load(kb + (int64_t)lane * HD + d, kk);
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
          for (int t = 0; t < 8; ++t) sc[h] += qs[h][d + t] * kk[t];
      }
    }
    const float scale = rsqrtf((float)HD);
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float sv = valid ? sc[h] * scale : -INFINITY;
      mw[h] = wave_max(sv);
      const float pv = valid ? __expf(sv - mw[h]) : 0.f;
      lw[h] = wave_sum(pv);
      ps[wave][h][lane] = pv;
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    const int nvalid = min(64, ctx - blk_pos);
#pragma unroll
    for (int t = 0; t < DPL; ++t) {
      const int d = lane * DPL + t;
      const T *vr = vb + (int64_t)d * KV_BLOCK;
      for (int pp = 0; pp < nvalid; pp += 8) {
        float vv[8];
        Vec8<T>::load(vr + pp, vv);
        // cache entries past the context are stale or uninitialised: never read them as numbers
#pragma unroll
        for (int u = 0; u < 8; ++u) vv[u] = (pp + u < nvalid) ? vv[u] : 0.f;
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
          for (int u = 0; u < 8; ++u) o[h][t] += ps[wave][h][pp + u] * vv[u];
      }
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      wm[wave][h] = mw[h];
      wl[wave][h] = lw[h];
    }
  }
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int t = 0; t < DPL; ++t) wo[wave][h][lane * DPL + t] = o[h][t];
  __syncthreads();

  // merge the four waves and write this split's partial
  for (int e = threadIdx.x; e < G * (HD + 2); e += 256) {
    const int h = e / (HD + 2), c = e % (HD + 2);
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, wm[w][h]);
    float acc = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (wm[w][h] == -INFINITY) continue;
      const float f = __expf(wm[w][h] - M);
      acc += f * (c < HD ? wo[w][h][c] : wl[w][h]);
    }
    float *dst = ws + (((int64_t)m * n_heads + g * G + h) * max_splits + s) * (HD + 2);
    dst[c] = (c == HD) ? M : acc;  // [0, HD): output, HD: max, HD + 1: sum
  }
}

// Merges a row's chunk partials for one query head: out = sum_s e^(m_s - M) o_s
// / sum_s e^(m_s - M) l_s with M the largest chunk maximum, taken in one pass
// with a running maximum; each thread owns one output dimension and issues
// the loads of eight chunks before it uses any.
template <typename T, int HD>
__global__ __launch_bounds__(HD) void decode_combine_kernel(RowMeta rows, int n_heads, int max_ctx,
                                                            int max_splits, const float *__restrict__ ws,
                                                            T *__restrict__ out) {
  constexpr int U = 8;
  const int h = blockIdx.x, m = blockIdx.y;
  const int c = threadIdx.x;
  const int ctx = min(rows.row_pos[m] + 1, max_ctx);
  const int ns = ctx > 0 ? (ctx + DEC_CHUNK - 1) / DEC_CHUNK : 0;
  const float *src = ws + ((int64_t)m * n_heads + h) * max_splits * (HD + 2);
  float M = -INFINITY, num = 0.f, den = 0.f;
  for (int s0 = 0; s0 < ns; s0 += U) {
    float mv[U], ov[U], lv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float *p = src + (int64_t)min(s0 + u, ns - 1) * (HD + 2);
      mv[u] = p[HD];
      ov[u] = p[c];
      lv[u] = p[HD + 1];
    }
    float nm = M;
#pragma unroll
    for (int u = 0; u < U; ++u) nm = fmaxf(nm, mv[u]);
    if (nm == -INFINITY) continue;
    const float r = __expf(M - nm);  // 0 while M is still -inf
    num *= r;
    den *= r;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float f = (s0 + u < ns) ? __expf(mv[u] - nm) : 0.f;
      num += f * ov[u];
      den += f * lv[u];
    }
    M = nm;
  }
  out[((int64_t)m * n_heads + h) * HD + c] = Act<T>::st(num / den);
}

// 16-bit decode attention on MFMA.  One wave owns one 64-position KV block:
// S = Q K^T is four 16x16 tiles (query heads of the group padded to 16 rows,
// positions as columns, head_dim as the contraction), the softmax is reduced
// across the 16 lanes that hold a row (DPP lane moves, no LDS), P goes through
// LDS into the A-operand
// layout, and O = P V contracts over positions with V read from its
// transposed [hd][64] block as 16-byte B fragments.  All K fragments of the
// block are requested before any is used, then all V fragments.
//
// FUSED: q is not read; the workgroup finishes the split-K QKV projection of
// its row first (QkvParts): the fp32 partials of its G query heads summed in
// split order and rotated into LDS, and in the workgroup of the row's last
// chunk the new K (rotated) and V entry of head g, written to the cache and
// put into the last block's fragments in place of what the cache held there.
// Its registers are bounded for four waves per SIMD (112 VGPRs, no spills):
// the 8B-shape decode step ran 75 us faster than with the separate finishing
// pass, against 41 us at the compiler's own three.
template <typename T, int HD, int G, bool FUSED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FUSED ? 4 : 1))) void decode_attn_mfma_kernel(
    const T *__restrict__ q, RowMeta rows, KVCache kv, int layer, int M, int n_heads, int max_ctx, int max_splits,
    float *__restrict__ ws, QkvParts qp) {
  typedef typename Mfma<T>::v8 v8;
  constexpr int KS = HD / 32;  // contraction steps over head_dim
  constexpr int NT = HD / 16;  // 16-wide output tiles over head_dim
  __shared__ T pls[4][16][64 + 8];
  __shared__ float wm[4][16], wl[4][16];
  __shared__ float wo[4][G][HD];
  __shared__ T qls[FUSED ? G : 1][HD];   // FUSED: the group's rotated q
  __shared__ T kvn[FUSED ? 2 : 1][HD];   // FUSED: the row's new K (rotated) and V entry
  // KV head fastest: consecutive block ids, which the dispatcher deals out
  // round-robin over the XCDs, are the heads of one work item
  const int g = blockIdx.x % kv.n_kv_heads;
  DecodeItem it;
  if (!decode_item(rows, M, max_ctx, blockIdx.x / kv.n_kv_heads, it)) return;
  const int m = it.m, s = it.s, slot = it.slot, ctx = it.ctx;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r16 = lane & 15, quad = lane >> 4, kq = quad * 8;
  const int blk_pos = s * DEC_CHUNK + wave * 64;
  const int nvalid = max(0, min(64, ctx - blk_pos));

  const int64_t base = nvalid > 0 ? kv_block_base(kv, layer, slot, blk_pos, g) : 0;
  v8 kf[4][KS];
  v8 qa[KS];
  // the row's new position, when it lies in this wave's block (FUSED)
  const int pnew = (FUSED && it.pos == ctx - 1) ? it.pos - blk_pos : -1;
  if constexpr (FUSED) {
    // Thread t takes q pair t of the group's heads and, in the workgroup of
    // the row's last chunk, pair t of head g's new K (t < HD/2) or V entry.
    // All their loads are issued before the K fragments' (the wait counter
    // is in order), so q is ready when K is.
    static_assert(G * HD / 2 <= 256, "one q pair per thread (decode_attention_fuses_qkv)");
    // Every load below is unconditional, at a clamped (valid) address, so
    // that the compiler issues them back to back and can wait for them
    // without waiting for the K fragments requested after them.
    const bool last = (s + 1) * DEC_CHUNK >= ctx && it.pos == ctx - 1;
    const int pos = it.pos, half = HD / 2, t = threadIdx.x;
    const int qdim = n_heads * HD, kvdim = kv.n_kv_heads * HD;
    const bool has_q = t < G * half, has_kv = last && t < HD, kv_k = t < half;
    const int tq = min(t, G * half - 1), iq = tq % half, hq = tq / half;
    const int nq = (g * G + hq) * HD + 2 * iq;
    const int tk = min(t, HD - 1), ik = tk % half;
    const int nkv = has_kv ? (kv_k ? qdim + g * HD + 2 * tk : qdim + kvdim + g * HD + 2 * (tk - half)) : nq;
    // all partials requested together (decode_attention_fuses_qkv: at most
    // DEC_QKV_SPLITS splits)
    constexpr int U = DEC_QKV_SPLITS;
    const float csq = qp.rope_cos[(int64_t)pos * half + iq], snq = qp.rope_sin[(int64_t)pos * half + iq];
    const float csk = qp.rope_cos[(int64_t)pos * half + ik], snk = qp.rope_sin[(int64_t)pos * half + ik];
    const int64_t kvo = kv_block_base(kv, layer, slot, pos, g);
    float2 pq[U], pk[U];
    float q0 = 0.f, q1 = 0.f, k0 = 0.f, k1 = 0.f;
#define DA_PARTS(s0)                                                                            \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                               \
    const int64_t r = (int64_t)min((s0) + u, qp.splits - 1) * M + m;                            \
    pq[u] = *(const float2 *)(qp.part + r * qp.N + nq);                                         \
    pk[u] = *(const float2 *)(qp.part + r * qp.N + nkv);                                        \
  }
// splits past the count add +0, which leaves every sum as it is (a sum that
// starts at +0 is never -0), and keeps each load's use unconditional
#define DA_SUM(s0)                                                                              \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                               \
    /* the partials are in registers here: no load is deferred into a branch */                 \
    asm volatile("" ::"v"(pq[u].x), "v"(pq[u].y), "v"(pk[u].x), "v"(pk[u].y));                  \
  }                                                                                             \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                               \
    const bool in_ = (s0) + u < qp.splits;                                                      \
    q0 += in_ ? pq[u].x : 0.f;                                                                  \
    q1 += in_ ? pq[u].y : 0.f;                                                                  \
    k0 += in_ ? pk[u].x : 0.f;                                                                  \
    k1 += in_ ? pk[u].y : 0.f;                                                                  \
  }
    DA_PARTS(0)
    {
      // this wave's K fragments, requested right behind the partials and
      // before the wait for them, so that the K round trip runs under the
      // partials' (the wait counter is in order: the partials can be waited
      // for with these still outstanding); unconditional (a wave without a
      // block reads the cache's first block, zeroed below)
      const T *kb = (const T *)kv.k + base;
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[nt][ks] = load8<T>(kb + (nt * 16 + r16) * HD + ks * 32 + kq);
    }
    DA_SUM(0)
#undef DA_PARTS
#undef DA_SUM
    if (nvalid <= 0) {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[nt][ks] = zero8<T>();
    }
    if (has_q) {
      float r0, r1;
      rope_rotate(q0, q1, csq, snq, r0, r1);
      qls[hq][iq] = Act<T>::st(r0);
      qls[hq][iq + half] = Act<T>::st(r1);
    }
    if (has_kv) {
      T *kc = (T *)kv.k + kvo + (int64_t)(pos % KV_BLOCK) * HD;
      T *vc = (T *)kv.v + kvo + pos % KV_BLOCK;
      if (kv_k) {
        float r0, r1;
        rope_rotate(k0, k1, csk, snk, r0, r1);
        const T t0 = Act<T>::st(r0), t1 = Act<T>::st(r1);
        kvn[0][ik] = t0;
        kvn[0][ik + half] = t1;
        kc[ik] = t0;
        kc[ik + half] = t1;
      } else {
        const int j = 2 * (tk - half);
        const T t0 = Act<T>::st(k0), t1 = Act<T>::st(k1);
        kvn[1][j] = t0;
        kvn[1][j + 1] = t1;
        vc[(int64_t)j * KV_BLOCK] = t0;
        vc[(int64_t)(j + 1) * KV_BLOCK] = t1;
      }
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qa[ks] = (r16 < G) ? load8<T>(&qls[r16][ks * 32 + kq]) : zero8<T>();
    if (pnew >= 0 && pnew < 64) {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
        if (nt * 16 + r16 == pnew) {
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) kf[nt][ks] = load8<T>(&kvn[0][ks * 32 + kq]);
        }
    }
  } else {
    const T *qrow = q + ((int64_t)m * n_heads + g * G + (r16 < G ? r16 : 0)) * HD;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qa[ks] = (r16 < G) ? load8<T>(qrow + ks * 32 + kq) : zero8<T>();
    if (nvalid > 0) {
      const T *kb = (const T *)kv.k + base;
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[nt][ks] = load8<T>(kb + (nt * 16 + r16) * HD + ks * 32 + kq);
    } else {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[nt][ks] = zero8<T>();
    }
  }
  floatx4_t sacc[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    sacc[nt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) sacc[nt] = Mfma<T>::m16(qa[ks], kf[nt][ks], sacc[nt]);
  }
  // V is requested once the K fragments are consumed: the registers K held
  // take V, which keeps the kernel at three workgroups per CU
  v8 vf[NT][2];
  if (nvalid > 0) {
    const T *vb = (const T *)kv.v + base;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) vf[nt][kk] = load8<T>(vb + (nt * 16 + r16) * KV_BLOCK + kk * 32 + kq);
  } else {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) vf[nt][0] = vf[nt][1] = zero8<T>();
  }
  // sacc[nt][i]: row (head) 4*quad + i, position nt*16 + r16
  const float scale = rsqrtf((float)HD);
  float mx[4], sm[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float v = -INFINITY;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const bool ok = nt * 16 + r16 < nvalid;
      sacc[nt][i] = ok ? sacc[nt][i] * scale : -INFINITY;
      v = fmaxf(v, sacc[nt][i]);
    }
    v = row16_max(v);
    mx[i] = v;
    float t = 0.f;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const float p = (v == -INFINITY) ? 0.f : __expf(sacc[nt][i] - v);
      sacc[nt][i] = p;
      t += p;
    }
    t = row16_sum(t);
    sm[i] = t;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) pls[wave][4 * quad + i][nt * 16 + r16] = Act<T>::st(sacc[nt][i]);
  }
  __syncthreads();
  v8 pa[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) pa[kk] = load8<T>(&pls[wave][r16][kk * 32 + kq]);
  // The V fragments are patched only now, after the softmax: a patch waits
  // for the fragments it edits, and placed right after their loads it held
  // the softmax of the wave (and, at the barrier above, its workgroup)
  // behind the V round trip.
  // Positions past the context hold stale or uninitialised cache entries.
  if (nvalid < 64) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (kk * 32 + kq + e >= nvalid) vf[nt][kk][e] = (typename Mfma<T>::v8){}[0];
  }
  // the row's new V entry (FUSED), in place of what the cache held there
  if (FUSED && pnew >= 0 && pnew < 64) {
    typedef __typeof__((typename Mfma<T>::v8){}[0]) elem_t;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const elem_t vn = __builtin_bit_cast(elem_t, kvn[FUSED ? 1 : 0][nt * 16 + r16]);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (kk * 32 + kq + e == pnew) vf[nt][kk][e] = vn;
    }
  }
  floatx4_t oacc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    oacc[nt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) oacc[nt] = Mfma<T>::m16(pa[kk], vf[nt][kk], oacc[nt]);
  }
  if (r16 == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      wm[wave][4 * quad + i] = mx[i];
      wl[wave][4 * quad + i] = sm[i];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int h = 4 * quad + i;
    if (h < G) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) wo[wave][h][nt * 16 + r16] = oacc[nt][i];
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < G * (HD + 2); e += 256) {
    const int h = e / (HD + 2), c = e % (HD + 2);
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, wm[w][h]);
    float acc = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (wm[w][h] == -INFINITY) continue;
      const float f = __expf(wm[w][h] - M);
      acc += f * (c < HD ? wo[w][h][c] : wl[w][h]);
    }
    float *dst = ws + (((int64_t)m * n_heads + g * G + h) * max_splits + s) * (HD + 2);
    dst[c] = (c == HD) ? M : acc;  // [0, HD): output, HD: max, HD + 1: sum
  }
}

template <typename T, int HD, int G>
static void launch_decode_group(dim3 grid, const T *q, const RowMeta &rows, const KVCache &kv, int layer, int M,
                                int n_heads, int max_ctx, int splits, float *ws, hipStream_t s, const QkvParts *qkv) {
  if constexpr (sizeof(T) == 2) {
    if constexpr (G * HD / 2 <= 256) {
      if (qkv) {
        decode_attn_mfma_kernel<T, HD, G, true><<<grid, 256, 0, s>>>(q, rows, kv, layer, M, n_heads, max_ctx, splits,
                                                                     ws, *qkv);
        return;
      }
    }
    decode_attn_mfma_kernel<T, HD, G, false><<<grid, 256, 0, s>>>(q, rows, kv, layer, M, n_heads, max_ctx, splits,
                                                                    ws, QkvParts{});
  } else {
    decode_attn_kernel<T, HD, G><<<grid, 256, 0, s>>>(q, rows, kv, layer, M, n_heads, max_ctx, splits, ws);
  }
}

template <typename T, int HD>
static void launch_decode_hd(const T *q, T *out, const RowMeta &rows, const KVCache &kv, int layer,
                             int M, int n_heads, int max_ctx, int items, float *ws, hipStream_t s,
                             const QkvParts *qkv) {
  const int G = n_heads / kv.n_kv_heads;
  if (qkv && !decode_attention_fuses_qkv(G, HD, qkv->splits)) return;
  const int splits = (max_ctx + DEC_CHUNK - 1) / DEC_CHUNK;
  if (items <= 0 || items > M * splits) items = M * splits;
  dim3 grid((unsigned)(items * kv.n_kv_heads));
  switch (G) {
    case 1: launch_decode_group<T, HD, 1>(grid, q, rows, kv, layer, M, n_heads, max_ctx, splits, ws, s, qkv); break;
    case 2: launch_decode_group<T, HD, 2>(grid, q, rows, kv, layer, M, n_heads, max_ctx, splits, ws, s, qkv); break;
    case 4: launch_decode_group<T, HD, 4>(grid, q, rows, kv, layer, M, n_heads, max_ctx, splits, ws, s, qkv); break;
    case 8: launch_decode_group<T, HD, 8>(grid, q, rows, kv, layer, M, n_heads, max_ctx, splits, ws, s, qkv); break;
    default: return;
  }
  decode_combine_kernel<T, HD><<<dim3(n_heads, M), HD, 0, s>>>(rows, n_heads, max_ctx, splits, ws, out);
}

template <typename T>
void launch_decode_attention(const T *q, T *out, const RowMeta &rows, const KVCache &kv, int layer,
                             int M, int n_heads, int max_ctx, int items, float *ws, hipStream_t s,
                             const QkvParts *qkv) {
  if (M <= 0) return;
  if (sizeof(T) != 2) qkv = nullptr;  // the fp32 path has no split QKV projection
  if (kv.head_dim == 128)
    launch_decode_hd<T, 128>(q, out, rows, kv, layer, M, n_heads, max_ctx, items, ws, s, qkv);
  else if (kv.head_dim == 64)
    launch_decode_hd<T, 64>(q, out, rows, kv, layer, M, n_heads, max_ctx, items, ws, s, qkv);
}

// ------------------------------------------------------------------ prefill

template <typename T, int HD>
__global__ __launch_bounds__(256) void prefill_attn_kernel(const T *__restrict__ q, T *__restrict__ out,
                                                           const int32_t *seq_start,
                                                           const int32_t *seq_slot, KVCache kv,
                                                           int layer, int n_heads) {
  constexpr int Q4 = HD / 4;  // dims per thread
  __shared__ T ks[64][HD + 2];
  __shared__ T vs[64][HD + 2];
  const int qt = blockIdx.x, h = blockIdx.y, j = blockIdx.z;
  const int row0 = seq_start[j];
  const int len = seq_start[j + 1] - row0;
  if (qt * 64 >= len) return;
  const int slot = seq_slot[j];
  const int g = h / (n_heads / kv.n_kv_heads);
  const int qi = threadIdx.x >> 2, qq = threadIdx.x & 3;
  const int qpos = qt * 64 + qi;
  const bool qvalid = qpos < len;
  float qv[Q4], o[Q4];
  const T *qr = q + ((int64_t)(row0 + (qvalid ? qpos : 0)) * n_heads + h) * HD + qq * Q4;
#pragma unroll
  for (int t = 0; t < Q4; ++t) {
    qv[t] = Act<T>::ld(qr[t]);
    o[t] = 0.f;
  }
  float mx = -INFINITY, l = 0.f;
  const float scale = rsqrtf((float)HD);
  const int last_key = min(len, qt * 64 + 64);  // keys [0, last_key)
  for (int kb = 0; kb * 64 < last_key; ++kb) {
    __syncthreads();
    const int64_t base = kv_block_base(kv, layer, slot, kb * 64, g);
    const T *kbp = (const T *)kv.k + base;
    const T *vbp = (const T *)kv.v + base;
    for (int e = threadIdx.x; e < 64 * HD; e += 256) {
      const int p = e / HD, d = e % HD;
      ks[p][d] = kbp[e];
      const int d2 = e / 64, p2 = e % 64;
      vs[p2][d2] = vbp[e];
    }
    __syncthreads();
    const int nk = min(64, last_key - kb * 64);
    for (int p = 0; p < nk; ++p) {
      float sc = 0.f;
#pragma unroll
      for (int t = 0; t < Q4; ++t) sc += qv[t] * Act<T>::ld(ks[p][qq * Q4 + t]);
      sc += __shfl_xor(sc, 1, 64);
      sc += __shfl_xor(sc, 2, 64);
      const int kpos = kb * 64 + p;
      if (kpos > qpos) continue;  // causal (uniform across the 4 threads of a row)
      sc *= scale;
      const float mn = fmaxf(mx, sc);
      const float corr = __expf(mx - mn);
      const float pe = __expf(sc - mn);
      l = l * corr + pe;
#pragma unroll
      for (int t = 0; t < Q4; ++t) o[t] = o[t] * corr + pe * Act<T>::ld(vs[p][qq * Q4 + t]);
      mx = mn;
    }
  }
  if (qvalid) {
    T *orow = out + ((int64_t)(row0 + qpos) * n_heads + h) * HD + qq * Q4;
    const float inv = 1.0f / l;
#pragma unroll
    for (int t = 0; t < Q4; ++t) orow[t] = Act<T>::st(o[t] * inv);
  }
}

// 16-bit causal prefill attention on MFMA (flash-attention style).  A
// workgroup owns 32 QW query rows of one (sequence, head), 32 to a wave, and
// walks the keys in blocks of 64.  Blocks are copied straight from the cache
// into LDS (two stages per key group: the next block lands while the current
// one is used), in the cache's own order (K [key][dim], V transposed
// [dim][key]) with the 16-byte pieces of a row XOR-swizzled, by choosing the
// address each lane copies from, so that the fragment reads below are free of
// bank conflicts.
//   S^T = K Q^T in 32x32x16 MFMAs: a lane holds one query's scores, so the
//   softmax's maximum and sum run in the lane's own registers and meet its
//   other half (lane ^ 32) once a block.  The K row that MFMA row i reads is i
//   with bits 2 and 3 swapped: then the eight probabilities a lane holds of
//   each 16 keys are consecutive keys, which is the B operand of
//   O^T += V^T P^T, and P never leaves the registers.
//   The running maximum is moved (and O and the sum rescaled) in the blocks
//   that raise it for one of the wave's rows, so that a row's largest
//   probability is exactly 1 before it is rounded to 16 bits.  Moving it only
//   where a score exceeds it by 2^8 ran 5% faster (three prompts around 2,100
//   tokens 298 against 313 us) and put the result 2.7% further from 64 bits
//   (three prompts of 900, bf16: 0.00206 against 0.00200).
// 32 rows a wave read half the LDS bytes per flop that 16 did (the 16-row
// kernel needed 256 B a clock and CU, all that LDS delivers), and the vector
// work of the softmax is what is left beside the MFMAs.  8B heads, fp16, 16-row
// waves against this kernel (in graphs of launches): one prompt of 300 tokens
// 12.0 -> 10.5 us, 547 19.0 -> 14.4, 1,300 42.9 -> 27.2, 4,096 252 -> 166 (830
// TFLOP/s, the clock down to 1.8 GHz); 8 prompts of 1,000 235 -> 106, 64 of 600
// 537 -> 372.  Deeper staging (three to five stages) and the next block's scores
// or the output products interleaved with the softmax by hand all measured the
// same or slower.
// KG key groups: group k of the waves takes every KG-th key block with its own
// stages, and the groups' (maximum, sum, O) meet in LDS at the end.
// Grid: x = head, dealt so that the heads of one KV head run on one XCD and
// share its L2; then with seq_major the query tiles and sequences, else the
// sequences and query tiles; tiles from the last, so that those with the most
// key blocks are dispatched first.
__device__ __forceinline__ float half_swap_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Rows of a sequence that are computed: as many as its row of the block table
// holds.  A tile of 128 rows can reach past max_len, by up to one block.
__device__ __forceinline__ int prefill_len(int len, const KVCache &kv) { return min(len, kv.max_blocks * KV_BLOCK); }
template <typename T>
__device__ __forceinline__ typename Mfma<T>::v8 pack8(const float *p) {
  typedef __typeof__((typename Mfma<T>::v8){}[0]) elem_t;
  typename Mfma<T>::v8 v;
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = (elem_t)p[j];
  return v;
}

// Stores a 32-dim tile of O^T times inv: a lane holds one row's dims 8 (r / 4) +
// 4 hh + r % 4.  The halves of the wave trade every other four dims, so that a
// lane stores eight consecutive dims at once (dst: the row's tile), from a base
// that is aligned for them; all lanes call, `valid` ones store.
template <typename T>
__device__ __forceinline__ void store_o32(T *dst, const floatx16_t &o, float inv, int hh, bool valid) {
  typedef uint32_t u4_t __attribute__((ext_vector_type(4), aligned(4)));
  const bool al4 = ((uintptr_t)dst & 3) == 0;
#pragma unroll
  for (int r8 = 0; r8 < 2; ++r8) {
    uint32_t w[2][2];  // dims 16 r8 + 8 i + 4 hh + {0, 1}, {2, 3}
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const T lo = Act<T>::st(o[r8 * 8 + i * 4 + e * 2] * inv), hi = Act<T>::st(o[r8 * 8 + i * 4 + e * 2 + 1] * inv);
        w[i][e] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | (uint32_t)__builtin_bit_cast(uint16_t, hi) << 16;
      }
    u4_t v;  // dims 16 r8 + 8 hh ..
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const auto t = __builtin_amdgcn_permlane32_swap(w[0][e], w[1][e], false, false);
      v[e] = t[0];
      v[e + 2] = t[1];
    }
    T *d = dst + r8 * 16 + hh * 8;
    if (valid) {
      if (al4) {
        *(u4_t *)d = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          d[2 * e] = __builtin_bit_cast(T, (uint16_t)v[e]);
          d[2 * e + 1] = __builtin_bit_cast(T, (uint16_t)(v[e] >> 16));
        }
      }
    }
  }
}

// Base-2 score past which the maximum is taken off before the scale: up to here
// a rounded mc is within 2^-13, which moves a weight of 1 by 8.5e-5, less than
// its rounding to 16 bits (2.4e-4 in f16).
constexpr float PFA_LARGE = 4096.f;

template <typename T, int HD, int QW, int KG>
__global__ __launch_bounds__(QW *KG * 64, 2) void prefill_attn_mfma_kernel(const T *__restrict__ q,
                                                                          T *__restrict__ out,
                                                                          const int32_t *seq_start,
                                                                          const int32_t *seq_slot, KVCache kv,
                                                                          int layer, int n_heads, int seq_major) {
  typedef typename Mfma<T>::v8 v8;
  constexpr int KS = HD / 16;            // contraction steps of S over head_dim
  constexpr int NT = HD / 32;            // 32-dim tiles of O^T
  constexpr int CK = HD / 8;             // 16-byte pieces of a K row
  constexpr int PB = 64 * HD * 2;        // bytes of a K (or V) block
  constexpr int STAGE = 2 * PB;
  constexpr int ND = PB / 1024 / QW;     // 1 KB copies per wave and block, K and V each
  __shared__ __attribute__((aligned(1024))) char lds[KG * 2 * STAGE];
  static_assert(QW * 64 >= HD, "a V row for every thread of a key group");
  static_assert(KG == 1 || (KG - 1) * QW * (NT * 16 + 2) * 256 <= KG * 2 * STAGE, "space of the group merge");
  const int xh = blockIdx.x;
  const int h = n_heads % 8 == 0 ? xh % 8 * (n_heads / 8) + xh / 8 : xh;
  const int qt = (int)(seq_major ? gridDim.y - 1 - blockIdx.y : gridDim.z - 1 - blockIdx.z);
  const int j = (int)(seq_major ? blockIdx.z : blockIdx.y);
  const int row0 = seq_start[j];
  const int len = prefill_len(seq_start[j + 1] - row0, kv);
  if (qt * QW * 32 >= len) return;
  const int slot = seq_slot[j];
  const int g = h / (n_heads / kv.n_kv_heads);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int kg = wave / QW, qw = wave % QW;
  const int l32 = lane & 31, hh = lane >> 5;
  const int q0 = qt * QW * 32 + qw * 32, qpos = q0 + l32;

  // Q^T as the B operand: this lane's query, dims 16 k + 8 hh ..
  v8 qb[KS];
  {
    const T *qr = q + ((int64_t)(row0 + min(qpos, len - 1)) * n_heads + h) * HD + hh * 8;
#pragma unroll
    for (int k = 0; k < KS; ++k) qb[k] = load8<T>(qr + k * 16);
  }
  const int nblk = min((qt * QW * 32 + QW * 32 + 63) / 64, (len + 63) / 64);  // causal: up to the diagonal
  const int nit = (nblk + KG - 1) / KG;

  // Byte offsets of the sequence's cache blocks (layer and head included): lane
  // i holds that of block win + i, and the wave reads them back with readlane.
  const int32_t *bt = kv.block_table + (int64_t)slot * kv.max_blocks;
  const int64_t head0 = ((int64_t)layer * kv.n_blocks * kv.n_kv_heads + g) * PB;
  const int64_t blk_step = (int64_t)kv.n_kv_heads * PB;
  int win = 0, off_lo, off_hi;
  auto window = [&]() __attribute__((always_inline)) {
    const int64_t off = head0 + bt[min(win + lane, nblk - 1)] * blk_step;
    off_lo = (int)off;
    off_hi = (int)(off >> 32);
    // used here, so that the wait for the load stands here and not at every
    // step's readlane
    asm volatile("" : "+v"(off_lo), "+v"(off_hi));
  };
  window();
  // Copies of this wave: K rows (1024 / (2 HD) a copy) and V rows (8 a copy);
  // lane l's 16 bytes land at piece l of the copy.
  constexpr int KR = 1024 / (HD * 2);
  const uint32_t lds0 = lds_addr(lds) + kg * 2 * STAGE + qw * ND * 1024;
  const int kcr = lane / CK, kcp = lane % CK, vcr = lane >> 3, vcp = lane & 7;
  auto swz = [](int row) __attribute__((always_inline)) { return CK == 16 ? row & 15 : (row >> 1) & 7; };
  uint32_t ko[ND], vo[ND];  // byte offsets inside a block
#pragma unroll
  for (int c = 0; c < ND; ++c) {
    const int n = qw * ND + c, kr = n * KR + kcr, vr = n * 8 + vcr;
    ko[c] = kr * HD * 2 + (kcp ^ swz(kr)) * 16;
    vo[c] = vr * KV_BLOCK * 2 + (vcp ^ ((vr >> 1) & 7)) * 16;
  }
  auto issue = [&](int it) __attribute__((always_inline)) {
    const int kb = it * KG + kg;
    if (kb >= nblk) return;
    if (kb >= win + 64) {
      win = kb;
      window();
    }
    const int64_t off = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(off_hi, kb - win) << 32) |
                                  (uint32_t)__builtin_amdgcn_readlane(off_lo, kb - win));
    const uint32_t st = lds0 + (it & 1) * STAGE;
#pragma unroll
    for (int c = 0; c < ND; ++c) {
      dma16s((const char *)kv.k + off, ko[c], st + c * 1024);
      dma16s((const char *)kv.v + off, vo[c], st + PB + c * 1024);
    }
  };

  floatx16_t o[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.f;
  // running maximum (raw scores), the score past which it moves, its base-2
  // value; this half's share of the sum
  float mref = -INFINITY, mc = 0.f, lsum = 0.f;
  bool large = false;  // wave-uniform: a row's |mc| is past PFA_LARGE
  const float c2 = rsqrtf((float)HD) * 1.44269504088896341f;
  // fragment addresses: K row with bits 2 and 3 swapped, V row l32 (+ 32 t)
  const int krow = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
  const int kfb = krow * HD * 2, kfx = (hh ^ swz(krow)) << 4;
  const int vfb = l32 * KV_BLOCK * 2, vfx = (hh ^ ((l32 >> 1) & 7)) << 4;

  issue(0);
  for (int it = 0; it < nit; ++it) {
    // this wave's copies of the block have landed; after the barrier everyone's
    // have, and the stage of the block before is free
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (it == nit - 1 && nblk * 64 > len) {
      // the sequence ends inside the last block: V entries past it are stale
      // or uninitialised, their weight is 0 but 0 * NaN is not.  The piece of a
      // row that the end falls into is masked, those behind it are cleared
      // without a read (a read, mask and write for every piece is a chain of
      // LDS round trips: one prompt of 100 tokens 7.2 us for 6.9).
      if ((nblk - 1) % KG == kg) {
        const int kvalid = len - (nblk - 1) * 64;
        char *vs = lds + kg * 2 * STAGE + (it & 1) * STAGE + PB;
        const int row = qw * 64 + lane;
        if (QW * 64 == HD || row < HD) {
          char *p = vs + row * KV_BLOCK * 2 + ((kvalid >> 3) ^ ((row >> 1) & 7)) * 16;
          u32x4_tt v = *(const u32x4_tt *)p;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const uint32_t lo = 2 * w < (kvalid & 7) ? 0xFFFFu : 0u;
            const uint32_t hi = 2 * w + 1 < (kvalid & 7) ? 0xFFFF0000u : 0u;
            v[w] &= (lo | hi);
          }
          *(u32x4_tt *)p = v;
        }
#pragma unroll
        for (int e = qw * 64 + lane; e < HD * 8; e += QW * 64) {
          const int r = e >> 3, key0 = ((e & 7) ^ ((r >> 1) & 7)) * 8;
          if (key0 > kvalid) *(u32x4_tt *)(vs + e * 16) = u32x4_tt{0, 0, 0, 0};
        }
      }
      __syncthreads();
    }
    if (it + 1 < nit) issue(it + 1);
    const int kb = it * KG + kg;
    if (kb >= nblk || kb * 64 > q0 + 31) continue;  // no block, or wholly past this wave's queries
    const char *ks = lds + kg * 2 * STAGE + (it & 1) * STAGE, *vs = ks + PB;
    floatx16_t s[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[t][r] = 0.f;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const v8 a = *(const v8 *)(ks + kfb + t * 32 * HD * 2 + (kfx ^ (k << 5)));
        s[t] = Mfma<T>::m32(a, qb[k], s[t]);
      }
    }
    // s[t][r]: key 32 t + 16 (r / 8) + 8 hh + r % 8 of the block
    if (kb * 64 + 63 > q0) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb * 64 + t * 32 + (r >> 3) * 16 + hh * 8 + (r & 7) > qpos) s[t][r] = -INFINITY;
    }
    float mx = s[0][0];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[t][r]);
    mx = half_swap_max(mx);
    if (__any(mx > mref)) {
      const float nm = fmaxf(mref, mx);
      const float corr = nm == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((mref - nm) * c2);
      mref = nm;
      mc = nm == -INFINITY ? 0.f : nm * c2;  // a row that has seen no key yet
      large = __any(fabsf(mc) > PFA_LARGE);
      lsum *= corr;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= corr;
    }
    // s c2 - mc in one FMA is off 0 at the maximum by what mc's rounding left
    // out, up to half a unit of mc: large scores have the maximum taken off
    // before the product instead
    float mo = mc;
    if (large) {
      const float m0 = mref == -INFINITY ? 0.f : mref;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[t][r] -= m0;
      mo = 0.f;
    }
    v8 pb[4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float p[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          p[r] = __builtin_amdgcn_exp2f(fmaf(s[t][u * 8 + r], c2, -mo));
          lsum += p[r];
        }
        pb[t * 2 + u] = pack8<T>(p);
      }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const v8 a = *(const v8 *)(vs + vfb + t * 32 * KV_BLOCK * 2 + (vfx ^ (k << 5)));
        o[t] = Mfma<T>::m32(a, pb[k], o[t]);
      }
  }
  if constexpr (KG > 1) {
    // groups 1.. hand (O, maximum, sum) to group 0, lane by lane
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    constexpr int REC = NT * 16 + 2;
    float *mrg = (float *)lds;
    if (kg > 0) {
      float *w = mrg + ((kg - 1) * QW + qw) * REC * 64 + lane;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) w[(t * 16 + r) * 64] = o[t][r];
      w[NT * 16 * 64] = mref;
      w[(NT * 16 + 1) * 64] = lsum;
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int k = 1; k < KG; ++k) {
      const float *w = mrg + ((k - 1) * QW + qw) * REC * 64 + lane;
      const float m1 = w[NT * 16 * 64], l1 = w[(NT * 16 + 1) * 64];
      const float nm = fmaxf(mref, m1);
      const float f0 = nm == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((mref - nm) * c2);
      const float f1 = nm == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m1 - nm) * c2);
      mref = nm;
      lsum = lsum * f0 + l1 * f1;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = o[t][r] * f0 + w[(t * 16 + r) * 64] * f1;
    }
  }
  // o[t][r]: dim 32 t + 8 (r / 4) + 4 hh + r % 4 of this lane's query
  const float inv = 1.0f / half_swap_sum(lsum);
  T *orow = out + ((int64_t)(row0 + qpos) * n_heads + h) * HD;
#pragma unroll
  for (int t = 0; t < NT; ++t) store_o32(orow + t * 32, o[t], inv, hh, qpos < len);
}

// Prompts of at most one cache block (64 tokens): a wave owns 32 query rows of a
// (sequence, head), with the products and layouts of the kernel above and
// nothing online in the softmax; queries 0..31 need the first 32 keys alone.
//   * STAGED: a workgroup is the two waves of a (sequence, head), with the block
//     copied into LDS once for both by whole 1 KB requests (the fragments ask
//     for 32 bytes of a row at a time, and memory bounds a step of many waves).
//   * Not STAGED, prompts of at most 32 tokens: one wave, which requests all its
//     K and V fragments straight from the cache at once; staging only adds a
//     barrier and LDS.
// The 128-row tiles above leave half the waves or more of such a prompt without
// a row.  8B heads, fp16, 64-row tiles of 16-row waves, those tiles, and these:
// 64 prompts of 16 tokens 19.5, 21.1 and 9.3 us; of 33 21.4, 23.8 and 15.3; of
// 64 25.7, 26.0 and 19.5; 16 of 60 8.0, 8.9 and 7.2; one prompt of 32 5.4, 5.4
// and 4.2.  40 heads of their own K and V, 64 prompts of 64: 29.8, 36.9 and 29.8.
template <typename T, int HD, bool STAGED>
__global__ __launch_bounds__(STAGED ? 128 : 64, 3) void prefill_attn_block_kernel(
    const T *__restrict__ q, T *__restrict__ out, const int32_t *seq_start, const int32_t *seq_slot, KVCache kv,
    int layer, int n_heads) {
  typedef typename Mfma<T>::v8 v8;
  constexpr int KS = HD / 16, NT = HD / 32, PB = 64 * HD * 2;
  __shared__ __attribute__((aligned(1024))) char lds[STAGED ? 2 * PB : 16];
  const int xh = blockIdx.x;
  // heads that share K and V on one XCD; else in the cache's order
  const int h = n_heads % 8 == 0 && n_heads > kv.n_kv_heads ? xh % 8 * (n_heads / 8) + xh / 8 : xh;
  const int j = blockIdx.y;
  const int qt = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row0 = seq_start[j];
  const int len = prefill_len(seq_start[j + 1] - row0, kv);
  if (len <= 0) return;
  const int64_t base = kv_block_base(kv, layer, seq_slot[j], 0, h / (n_heads / kv.n_kv_heads));
  const T *kb = (const T *)kv.k + base, *vb = (const T *)kv.v + base;
  const int l32 = lane & 31, hh = lane >> 5, qpos = qt * 32 + l32;
  const int krow = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
  // 16-byte pieces of K and V rows are XOR-swizzled in LDS, as above
  constexpr int CK = HD / 8, KR = 1024 / (HD * 2);
  auto swz = [](int row) __attribute__((always_inline)) { return CK == 16 ? row & 15 : (row >> 1) & 7; };
  if constexpr (STAGED) {
    const uint32_t lds0 = lds_addr(lds);
#pragma unroll
    for (int c = 0; c < PB / 2048; ++c) {
      const int n = qt * (PB / 2048) + c, kr = n * KR + lane / CK, vr = n * 8 + (lane >> 3);
      // copies of keys past the sequence alone are left out: masked below
      if (n * KR < len) dma16s(kb, kr * HD * 2 + ((lane % CK) ^ swz(kr)) * 16, lds0 + n * 1024);
      dma16s(vb, vr * KV_BLOCK * 2 + ((lane & 7) ^ ((vr >> 1) & 7)) * 16, lds0 + PB + n * 1024);
    }
  }
  const T *qr = q + ((int64_t)(row0 + min(qpos, len - 1)) * n_heads + h) * HD + hh * 8;
  v8 qb[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) qb[k] = load8<T>(qr + k * 16);
  if constexpr (STAGED) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  auto rows = [&](auto tiles) __attribute__((always_inline)) {
    constexpr int TK = decltype(tiles)::value;  // 32-key tiles
    v8 ka[KS], va[2][NT];
    if constexpr (!STAGED) {
#pragma unroll
      for (int k = 0; k < KS; ++k) ka[k] = load8<T>(kb + krow * HD + k * 16 + hh * 8);
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int t = 0; t < NT; ++t) va[k][t] = load8<T>(vb + (t * 32 + l32) * KV_BLOCK + k * 16 + hh * 8);
    }
    floatx16_t s[TK];
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < TK; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[t][r] = 0.f;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        v8 a;
        if constexpr (STAGED) a = *(const v8 *)(lds + (t * 32 + krow) * HD * 2 + (((hh ^ swz(krow)) << 4) ^ (k << 5)));
        else a = ka[k];
        s[t] = Mfma<T>::m32(a, qb[k], s[t]);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (t * 32 + (r >> 3) * 16 + hh * 8 + (r & 7) > qpos) s[t][r] = -INFINITY;
        mx = fmaxf(mx, s[t][r]);
      }
    }
    mx = half_swap_max(mx);
    const float m0 = mx == -INFINITY ? 0.f : mx, c2 = rsqrtf((float)HD) * 1.44269504088896341f;
    float lsum = 0.f;
    v8 pb[TK * 2];
    // V entries past the sequence are stale or uninitialised: their weight is 0
    // but 0 * NaN is not
    u32x4_tt keep[TK * 2];
#pragma unroll
    for (int k = 0; k < TK * 2; ++k) {
      float p[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        p[r] = __builtin_amdgcn_exp2f((s[k >> 1][(k & 1) * 8 + r] - m0) * c2);
        lsum += p[r];
      }
      pb[k] = pack8<T>(p);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int key = k * 16 + hh * 8 + 2 * w;
        keep[k][w] = (key < len ? 0xFFFFu : 0u) | (key + 1 < len ? 0xFFFF0000u : 0u);
      }
    }
    const float inv = 1.0f / half_swap_sum(lsum);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      floatx16_t o;
#pragma unroll
      for (int r = 0; r < 16; ++r) o[r] = 0.f;
#pragma unroll
      for (int k = 0; k < TK * 2; ++k) {
        u32x4_tt v;
        if constexpr (STAGED)
          v = *(const u32x4_tt *)(lds + PB + (t * 32 + l32) * KV_BLOCK * 2 +
                                  (((hh ^ ((l32 >> 1) & 7)) << 4) ^ (k << 5)));
        else
          v = __builtin_bit_cast(u32x4_tt, va[k][t]);
        o = Mfma<T>::m32(__builtin_bit_cast(v8, v & keep[k]), pb[k], o);
      }
      store_o32(out + ((int64_t)(row0 + qpos) * n_heads + h) * HD + t * 32, o, inv, hh, qpos < len);
    }
  };
  if (qt == 0) {
    rows(std::integral_constant<int, 1>());
  } else if constexpr (STAGED) {
    if (len > 32) rows(std::integral_constant<int, 2>());
  }
}

// Steps of at most this many prompts dispatch the longest query tiles of all
// prompts first; with more, each prompt's tiles run together, so that its keys
// and values stay in the L2.
constexpr int PF_ATTN_LONGEST_FIRST_MAX_SEQ = 4;
template <typename T, int HD, int QW, int KG>
static void launch_prefill_mfma(const T *q, T *out, const int32_t *seq_start, const int32_t *seq_slot, int n_seq,
                                int max_len, const KVCache &kv, int layer, int n_heads, hipStream_t s) {
  const int tiles = (max_len + QW * 32 - 1) / (QW * 32);
  const int seq_major = n_seq > PF_ATTN_LONGEST_FIRST_MAX_SEQ;
  const dim3 grid = seq_major ? dim3(n_heads, tiles, n_seq) : dim3(n_heads, n_seq, tiles);
  prefill_attn_mfma_kernel<T, HD, QW, KG><<<grid, QW * KG * 64, 0, s>>>(q, out, seq_start, seq_slot, kv, layer,
                                                                         n_heads, seq_major);
}

template <typename T, int HD>
static void launch_prefill_hd(const T *q, T *out, const int32_t *seq_start, const int32_t *seq_slot, int n_seq,
                              int max_len, const KVCache &kv, int layer, int n_heads, hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    // Prompts of one cache block have kernels of their own (figures there).
    // Two key groups for one prompt whose workgroups use half the CUs or more
    // and would fit two to every CU: each CU's second set of waves then comes
    // from the key groups, and the longest tile walks half its blocks (8B heads,
    // one group against two: 400 tokens, 128 workgroups, 12.8 against 12.3 us;
    // 547, 160, 15.6 against 14.3; 1,300, 352, 32.7 against 27.2; 2,048, 512,
    // 55.0 against 48.8).  Below, the merge costs what it saves (384 tokens, 96:
    // 12.2 against 12.0; 256, 64: 9.5 against 10.0); above, two workgroups a CU
    // overlap better (2,300 tokens, 576: 64.6 against 66.4; 2,600, 672: 76
    // against 83).  40 heads of their own K and V: 480 workgroups 42.7 against
    // 40.2, 520 47.3 against 48.4.  64 heads, 8 of K and V, gain least: 640
    // tokens, 320, 19.3 against 17.7; 700, 384, 20.7 against 21.6; 1,000, 512,
    // 31.0 against 30.7.  With several prompts the grid's upper bound says
    // little about the live tiles (3 x 400 tokens: 16.5 against 19.2).
    const int64_t wgs = (int64_t)((max_len + 127) / 128) * n_heads;
    if ((((uintptr_t)kv.k | (uintptr_t)kv.v) & 15) == 0) {
      if (max_len <= 32)
        prefill_attn_block_kernel<T, HD, false><<<dim3(n_heads, n_seq), 64, 0, s>>>(q, out, seq_start, seq_slot, kv,
                                                                                    layer, n_heads);
      else if (max_len <= KV_BLOCK)
        prefill_attn_block_kernel<T, HD, true><<<dim3(n_heads, n_seq), 128, 0, s>>>(q, out, seq_start, seq_slot, kv,
                                                                                    layer, n_heads);
      else if (n_seq == 1 && wgs >= 128 && wgs <= 512)
        launch_prefill_mfma<T, HD, 4, 2>(q, out, seq_start, seq_slot, n_seq, max_len, kv, layer, n_heads, s);
      else
        launch_prefill_mfma<T, HD, 4, 1>(q, out, seq_start, seq_slot, n_seq, max_len, kv, layer, n_heads, s);
      return;
    }
  }
  // fp32, and 16-bit caches off 16 bytes (the kernels above read and copy whole
  // 16-byte pieces of them)
  const dim3 grid((max_len + 63) / 64, n_heads, n_seq);
  prefill_attn_kernel<T, HD><<<grid, 256, 0, s>>>(q, out, seq_start, seq_slot, kv, layer, n_heads);
}

template <typename T>
void launch_prefill_attention(const T *q, T *out, const int32_t *seq_start, const int32_t *seq_slot,
                              int n_seq, int max_len, const KVCache &kv, int layer, int n_heads,
                              hipStream_t s) {
  if (n_seq <= 0) return;
  if (kv.head_dim == 128)
    launch_prefill_hd<T, 128>(q, out, seq_start, seq_slot, n_seq, max_len, kv, layer, n_heads, s);
  else if (kv.head_dim == 64)
    launch_prefill_hd<T, 64>(q, out, seq_start, seq_slot, n_seq, max_len, kv, layer, n_heads, s);
}

#define INST(T)                                                                                     \
  template void launch_decode_attention<T>(const T *, T *, const RowMeta &, const KVCache &, int,   \
                                           int, int, int, int, float *, hipStream_t,                \
                                           const QkvParts *);                                       \
  template void launch_prefill_attention<T>(const T *, T *, const int32_t *, const int32_t *, int, \
                                            int, const KVCache &, int, int, hipStream_t);
INST(float)
INST(bf16_t)
INST(f16_t)
#undef INST

}  // namespace lp
