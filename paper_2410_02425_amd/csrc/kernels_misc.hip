// Embedding gather, RMSNorm (with split-K residual folding), greedy argmax and
// the device-side weight generator.
#include <type_traits>

#include "device.hpp"

namespace lp {

// ------------------------------------------------------------------ embedding

// One workgroup per row.  The row is read in 16-byte pieces, four per thread
// requested before any is stored, so a row of up to 4,096 16-bit (2,048
// fp32) values costs one memory round trip; rows whose length is not a
// multiple of the piece take the element loop.  A row of logits that holds
// nothing but NaN has no largest one, and its token (argmax_kernel's 0x7fffffff)
// is outside the vocabulary: such a token embeds as NaN, without a read.
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(const T *__restrict__ E, const int32_t *pool,
                                                    const int32_t *tok_idx, const int32_t *row_slot,
                                                    const int32_t *slot_tok, float *__restrict__ x,
                                                    int d, int V) {
  const int m = blockIdx.x;
  const int ti = tok_idx[m];
  const int tok = ti >= 0 ? pool[ti] : slot_tok[row_slot[m]];
  float *dst = x + (int64_t)m * d;
  if ((uint32_t)tok >= (uint32_t)V) {
    for (int c = threadIdx.x; c < d; c += blockDim.x) dst[c] = NAN;
    return;
  }
  const T *src = E + (int64_t)tok * d;
  constexpr int EV = 16 / sizeof(T);  // elements per 16-byte piece
  constexpr int U = 4;
  if (d % EV == 0) {
    const int nv = d / EV;
    for (int c0 = threadIdx.x; c0 < nv; c0 += 256 * U) {
      uint4 r[U];
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = ((const uint4 *)src)[min(c0 + u * 256, nv - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * 256;
        if (c < nv) {
          const T *e = (const T *)&r[u];
#pragma unroll
          for (int k = 0; k < EV; k += 4)
            *(float4 *)(dst + (int64_t)c * EV + k) =
                make_float4(Act<T>::ld(e[k]), Act<T>::ld(e[k + 1]), Act<T>::ld(e[k + 2]), Act<T>::ld(e[k + 3]));
        }
      }
    }
  } else {
    for (int c = threadIdx.x; c < d; c += blockDim.x) dst[c] = Act<T>::ld(src[c]);
  }
}

template <typename T>
void launch_embed(const T *E, const int32_t *pool, const int32_t *tok_idx, const int32_t *row_slot,
                  const int32_t *slot_tok, float *x, int M, int d, int V, hipStream_t s) {
  if (M <= 0) return;
  embed_kernel<T><<<M, 256, 0, s>>>(E, pool, tok_idx, row_slot, slot_tok, x, d, V);
}

// ------------------------------------------------------------------ RMSNorm

// One workgroup per row.  The residual row, every split-K partial of it and
// the gains are requested before any is used (NP is the partial count), so a
// row costs one memory latency rather than one per partial.  V4 float4 per
// thread: one for rows of up to 4,096, two up to 8,192, with d / (4 V4)
// threads (rounded to waves).  A 64 x 4,096 fold of eight partials took
// 4.2 us on 1,024 threads against 10.9 us on 256 with four float4 each
// (harness, partials cold): more waves keep more of the row in flight.
template <typename T, int NP, int V4>
__global__ __launch_bounds__(1024) void rmsnorm_kernel(float *x, const float *part, int64_t part_stride,
                                                       const int32_t *rows, const float *__restrict__ g,
                                                       T *__restrict__ y, int d, float eps) {
  __shared__ float red[16];
  const int j = blockIdx.x;
  const int src = rows ? rows[j] : j;
  const int d4 = d >> 2;
  const int nt = blockDim.x;
  float4 *xr = (float4 *)(x + (int64_t)src * d);
  const float4 *g4 = (const float4 *)g;
  float4 v[V4], gv[V4];
  float4 p[NP > 0 ? NP : 1][V4];
#pragma unroll
  for (int e = 0; e < V4; ++e) {
    const int c = threadIdx.x + e * nt;
    if (c < d4) {
      v[e] = xr[c];
      gv[e] = g4[c];
#pragma unroll
      for (int s = 0; s < NP; ++s) p[s][e] = ((const float4 *)(part + s * part_stride + (int64_t)src * d))[c];
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int e = 0; e < V4; ++e) {
    const int c = threadIdx.x + e * nt;
    if (c < d4) {
#pragma unroll
      for (int s = 0; s < NP; ++s) {
        v[e].x += p[s][e].x;
        v[e].y += p[s][e].y;
        v[e].z += p[s][e].z;
        v[e].w += p[s][e].w;
      }
      if (NP) xr[c] = v[e];
      ss += v[e].x * v[e].x + v[e].y * v[e].y + v[e].z * v[e].z + v[e].w * v[e].w;
    }
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < (nt >> 6); ++w) tot += red[w];
  const float r = rsqrtf(tot / (float)d + eps);
  T *yr = y + (int64_t)j * d;
#pragma unroll
  for (int e = 0; e < V4; ++e) {
    const int c = threadIdx.x + e * nt;
    if (c < d4) {
      const float4 gg = gv[e];
      yr[4 * c + 0] = Act<T>::st(v[e].x * r * gg.x);
      yr[4 * c + 1] = Act<T>::st(v[e].y * r * gg.y);
      yr[4 * c + 2] = Act<T>::st(v[e].z * r * gg.z);
      yr[4 * c + 3] = Act<T>::st(v[e].w * r * gg.w);
    }
  }
}

template <typename T>
void launch_rmsnorm(float *x, const float *part, int n_part, int64_t part_stride, const int32_t *rows,
                    const float *g, T *y, int M, int d, float eps, hipStream_t s) {
  if (M <= 0) return;
  // whole waves, V4 float4 per thread (d <= 8192)
  const int v4 = d / 4 <= 1024 ? 1 : 2;
  const int threads = std::min(1024, std::max(64, ((d / (4 * v4)) + 63) / 64 * 64));
#define NORM_CASE(NPV)                                                                                  \
  case NPV:                                                                                             \
    if (v4 == 1)                                                                                        \
      rmsnorm_kernel<T, NPV, 1><<<M, threads, 0, s>>>(x, part, part_stride, rows, g, y, d, eps);        \
    else                                                                                                \
      rmsnorm_kernel<T, NPV, 2><<<M, threads, 0, s>>>(x, part, part_stride, rows, g, y, d, eps);        \
    break;
  switch (n_part) {
    NORM_CASE(0) NORM_CASE(1) NORM_CASE(2) NORM_CASE(3) NORM_CASE(4) NORM_CASE(5) NORM_CASE(6)
    NORM_CASE(7) NORM_CASE(8) NORM_CASE(9) NORM_CASE(10) NORM_CASE(11) NORM_CASE(12)
    NORM_CASE(13) NORM_CASE(14) NORM_CASE(15) NORM_CASE(16)
    default: break;  // callers never pass more than 16 partials
  }
#undef NORM_CASE
}

// ------------------------------------------------------------------ argmax

// Walks over a row of logits (argmax and sampling).  A workgroup of ROW_W
// waves owns a row and each wave a contiguous part of it, ROW_STEP elements a
// step (16 bytes a lane) and eight steps' loads requested before any is used,
// so a 128,256-entry row costs four memory round trips.  One CU's vector
// units, not its loads, bound such a pass (a row is 2,004 wave instructions
// for every instruction an element takes, 0.8 us on four SIMDs), so a full
// batch of steps runs without bounds checks.  The loads ask for the alignment
// of a float only, which is all that a 16-byte global load needs, so rows of
// any stride take them.
constexpr int ROW_W = 16, ROW_T = ROW_W * 64, ROW_STEP = 256, ROW_U = 8, ROW_UT = 2;
struct RowPart {
  const float *row;
  int beg, end;  // this wave's elements
};
__host__ __device__ inline int row_chunk(int V) { return (V + ROW_W * ROW_STEP - 1) / (ROW_W * ROW_STEP) * ROW_STEP; }
__device__ __forceinline__ RowPart row_part(const float *logits, int64_t ld, int m, int V) {
  const int chunk = row_chunk(V), w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int beg = min(V, w * chunk);
  return {logits + (int64_t)m * ld, beg, min(V, beg + chunk)};
}
__device__ __forceinline__ float4 row_load16(const float *p) {
  typedef float f4_t __attribute__((ext_vector_type(4), aligned(4)));
  const f4_t v = *(const f4_t *)p;
  return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ float4 row_load4(const RowPart &R, int c, float fill) {
  float4 v;
  v.x = c < R.end ? R.row[c] : fill;
  v.y = c + 1 < R.end ? R.row[c + 1] : fill;
  v.z = c + 2 < R.end ? R.row[c + 2] : fill;
  v.w = c + 3 < R.end ? R.row[c + 3] : fill;
  return v;
}
// f(index of the first element, four logits, how many of them exist) for this
// lane's elements, g(batch) after every ROW_U steps.  All lanes are active in
// every call.
template <typename F, typename G>
__device__ __forceinline__ void row_walk(const RowPart &R, F f, G g) {
  const int lane = threadIdx.x & 63;
  int batch = 0;
  for (int c0 = R.beg; c0 < R.end; c0 += ROW_U * ROW_STEP, ++batch) {
    if (c0 + ROW_U * ROW_STEP <= R.end) {
      float4 v[ROW_U];
#pragma unroll
      for (int u = 0; u < ROW_U; ++u) v[u] = row_load16(R.row + c0 + u * ROW_STEP + lane * 4);
#pragma unroll
      for (int u = 0; u < ROW_U; ++u) f(c0 + u * ROW_STEP + lane * 4, v[u], std::integral_constant<int, 4>());
    } else {
      // the last steps, two in flight (four spill the sampler's registers): the
      // same loads, held to the row's last whole piece, and a piece that the
      // row ends in by elements.  Loaded by elements one step at a time, argmax
      // of 64 x 20,000 took 7.2 us for 3.7, of 50,257 (rows off 16 bytes) 13.8
      // for 4.8.
#pragma unroll 1
      for (int c1 = c0; c1 < R.end; c1 += ROW_UT * ROW_STEP) {
        float4 v[ROW_UT];
        if (R.end >= 4) {
#pragma unroll
          for (int u = 0; u < ROW_UT; ++u) v[u] = row_load16(R.row + min(c1 + u * ROW_STEP + lane * 4, R.end - 4));
        }
#pragma unroll
        for (int u = 0; u < ROW_UT; ++u) {
          const int c = c1 + u * ROW_STEP + lane * 4;
          if (c + 4 > R.end) v[u] = row_load4(R, c, -INFINITY);
          f(c, v[u], min(4, max(0, R.end - c)));
        }
      }
    }
    g(batch);
  }
}
// This lane's largest logit, where its first 16-byte piece that holds it
// starts, and whether it met a NaN (which no comparison picks).
struct RowBest {
  float v;
  int c;
  bool nan;
};
__device__ __forceinline__ RowBest row_best(const RowPart &R) {
  RowBest b{-INFINITY, R.beg, false};
  row_walk(
      R,
      [&](int c, const float4 &v, auto) {
        const float m = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
        b.nan |= __builtin_isunordered(v.x, v.y) | __builtin_isunordered(v.z, v.w);
        if (m > b.v) {
          b.v = m;
          b.c = c;
        }
      },
      [](int) {});
  return b;
}
// The row's largest logit, in every thread.
__device__ __forceinline__ float row_max(const RowBest &b, float (&red)[ROW_W]) {
  const float w = wave_max(b.v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
  __syncthreads();
  return row16_max(red[threadIdx.x & (ROW_W - 1)]);
}
// The lowest index that holds mx (0x7fffffff: none, a row of NaN only), in
// every thread.
__device__ __forceinline__ int row_first(const RowPart &R, const RowBest &b, float mx, int (&red)[ROW_W]) {
  int idx = 0x7fffffff;
  if (mx == -INFINITY) {
    for (int c = R.beg + (int)(threadIdx.x & 63); c < R.end; c += 64)
      if (R.row[c] == mx) {
        idx = c;
        break;
      }
  } else if (b.v == mx) {
#pragma unroll
    for (int e = 3; e >= 0; --e)
      if (b.c + e < R.end && R.row[b.c + e] == mx) idx = b.c + e;
  }
  idx = (int)wave_min_u32((uint32_t)idx);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = idx;
  __syncthreads();
  return (int)wave_min_u32((uint32_t)red[threadIdx.x & (ROW_W - 1)]);
}

// One workgroup per row: the maximum, then the lowest index that holds it,
// found again in the one piece its lane remembers.  64 rows of 128,256: 15.5
// -> 8.0 us (an index was merged with every element before).
__global__ __launch_bounds__(ROW_T) void argmax_kernel(const float *__restrict__ logits, int64_t ld, int V,
                                                       const int32_t *out_slot, int32_t *slot_tok, int32_t *tok_log) {
  __shared__ float sv[ROW_W];
  __shared__ int si[ROW_W];
  const int m = blockIdx.x;
  const RowPart R = row_part(logits, ld, m, V);
  const RowBest b = row_best(R);
  const int bi = row_first(R, b, row_max(b, sv), si);
  if (threadIdx.x == 0) {
    if (out_slot) slot_tok[out_slot[m]] = bi;
    tok_log[m] = bi;
  }
}

void launch_argmax(const float *logits, int64_t ld, int M, int V, const int32_t *out_slot, int32_t *slot_tok,
                   int32_t *tok_log, hipStream_t s) {
  if (M <= 0) return;
  argmax_kernel<<<M, ROW_T, 0, s>>>(logits, ld, V, out_slot, slot_tok, tok_log);
}

// ------------------------------------------------------------------ weight generator

// Philox4x32 with ten rounds (Salmon et al., SC'11).
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t lo0 = 0xD2511F53u * c[0], hi0 = __umulhi(0xD2511F53u, c[0]);
    const uint32_t lo1 = 0xCD9E8D57u * c[2], hi1 = __umulhi(0xCD9E8D57u, c[2]);
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
  }
}

// ------------------------------------------------------------------ sampling

// Non-greedy next-token choice per row (the sampling parameters carried by
// requests, Sec. III-A).  Every decision after the per-token weights is exact
// integer arithmetic, so the result does not depend on reduction order:
//  * temperature <= 0 or top_p <= 0: greedy (lowest index among maxima);
//  * candidates: all tokens, or with 0 < top_k < V those whose logit is at
//    least the top_k-th largest logit (ties at it kept), found by a radix
//    select over order-preserving integer keys of the logits;
//  * weight of a candidate: q = floor(exp((logit - max) / T) * 2^40);
//  * top_p < 1: with Z the candidates' total weight and
//    need = ceil(Z * floor(top_p * 2^24) / 2^24), keep the candidates whose q
//    is at least t, the largest value whose heavier-or-equal candidates sum to
//    at least need (a radix descent over q with 64-bit mass histograms);
//  * draw: u24 = the first Philox4x32-10 output word (key, counter as given)
//    shifted right by 8; r = floor(Z_kept * u24 / 2^24); the token is the kept
//    candidate, in vocabulary order, whose cumulative weight interval holds r.
// One workgroup per row; vector work per element bounds it (see the walk
// above), so the row is passed over as few times as the parameters allow:
//  * the maximum, each lane's own maximum kept;
//  * top_k <= SP_FASTK: at least top_k lanes hold a maximum of at least L, the
//    top_k-th largest of them to within a histogram bin, so only the lanes
//    that reach L hold candidates and only those read their elements again;
//    larger top_k, rows with a NaN and rows whose list overflows select on
//    histograms over the whole row;
//  * no top_p: one pass adds up weights per 2,048 elements (a piece), which
//    gives the total and, by a scan, the piece that holds the draw;
//  * top_p: one pass for the total and the masses of log-scale weight bins,
//    one that adds up the pieces of everything heavier than the chosen bin and
//    lists that bin's elements, which the remaining levels refine in LDS.
// Candidate sets of at most SP_SMALL are settled by direct sums.  64 rows of
// 128,256 logits, in a graph of launches, against five passes with an index
// merge, an atomic or a 64-bit shuffle an element: greedy 23.4 -> 9.0 us,
// temperature 82.7 -> 25.5, top-k 40 68.2 -> 27.4, top-p 0.9 157 -> 74.4, top-k 50
// with top-p 0.95 90.8 -> 32.9.
// Keys in the order of the values: x + 0 makes the zeros of either sign one key,
// as they are one value to the float comparisons that choose a lane's maximum.
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t b = __float_as_uint(x + 0.0f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// A weight before and after the floor.
__device__ __forceinline__ float f_weight(float l, float mx, float inv_t) {
  return __expf((l - mx) * inv_t) * 1099511627776.0f;  // 2^40; exp <= 1
}
__device__ __forceinline__ uint64_t q_weight(float l, float mx, float inv_t) {
  return (uint64_t)f_weight(l, mx, inv_t);
}

// (a * b) >> 24 for a < 2^58, b < 2^25, rounded up when `up`
__device__ __forceinline__ uint64_t mul_shift24(uint64_t a, uint64_t b, bool up) {
  const uint64_t lo = a * b, hi = __umul64hi(a, b);
  uint64_t r = (hi << 40) | (lo >> 24);
  if (up && (lo & 0xFFFFFFull)) ++r;
  return r;
}

constexpr int SP_T = ROW_T;    // threads per row
constexpr int SP_NB = 2048;    // bins of a radix level (11 bits)
constexpr int SP_CAP = 8192;   // values held in LDS after a compaction
constexpr int SP_DRAW = 1024;  // kept candidates drawn in LDS (one per thread)
constexpr int SP_FASTK = 512;  // largest top_k selected through the lanes' maxima
constexpr int SP_SMALL = 256;  // candidates settled by direct sums over the list
constexpr int SP_PIECE = ROW_U * ROW_STEP;  // elements per piece of the draw: one batch of a wave
static_assert((int64_t)SP_T * SP_PIECE >= SAMPLE_MAX_V && SAMPLE_MAX_V % (ROW_W * SP_PIECE) == 0,
              "one piece of the draw per thread");

struct SampleLds {
  uint64_t hist[SP_NB];
  uint64_t lv[SP_CAP];     // order key or weight of a listed element
  int32_t li[SP_CAP];      // its vocabulary index
  uint64_t cq[SP_DRAW];    // candidates of an LDS draw: weight
  int32_t ci[SP_DRAW];     // ... and index
  uint64_t pm[SP_T];       // kept mass per piece
  uint64_t red[16];
  uint64_t sel[4];
  float fmax[ROW_W];
  int imax[ROW_W];
  uint32_t kred[ROW_W];
  int n_list, n_cand, found, pick;
};

__device__ __forceinline__ float key_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// inclusive scan of v over the block's threads (thread order), and the total
__device__ uint64_t sp_scan(uint64_t v, uint64_t *red, uint64_t &total) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const uint64_t x = wave_scan(v);
  __syncthreads();
  if (lane == 63) red[w] = x;
  __syncthreads();
  const uint64_t waves = row16_scan(red[lane & 15]);
  total = readlane_u64(waves, 15);
  return x + (w ? readlane_u64(waves, w - 1) : 0);
}

// Radix level selection over hist[0..nb): the largest bin b >= 1 whose mass
// from the top (plus `above`) reaches need, else 0 -- the bin where a walk
// down from the highest bin first reaches need.  Writes sel[0] = mass above
// b (plus above), sel[1] = b, sel[2] = sel[0] + hist[b].  Thread t owns bins
// nb-1-2t and nb-2-2t.
__device__ void sp_select(SampleLds &S, int nb, uint64_t need, uint64_t above) {
  const int t = threadIdx.x;
  const int hi = nb - 1 - 2 * t, lo = hi - 1;
  const uint64_t hh = (t < nb / 2) ? S.hist[hi] : 0, hl = (t < nb / 2) ? S.hist[lo] : 0;
  uint64_t total;
  const uint64_t incl = sp_scan(hh + hl, S.red, total);
  const uint64_t excl = incl - hh - hl;
  if (t == 0) S.pick = 0;
  __syncthreads();
  if (t < nb / 2) {
    int b = -1;
    if (above + excl + hh >= need && hi >= 1) b = hi;
    else if (above + incl >= need && lo >= 1) b = lo;
    if (b >= 0) atomicMax(&S.pick, b);
  }
  __syncthreads();
  const int b = S.pick;
  if (t < nb / 2 && (b == hi || b == lo)) {
    const uint64_t a = above + excl + (b == lo ? hh : 0);
    S.sel[0] = a;
    S.sel[1] = (uint64_t)b;
    S.sel[2] = a + (b == lo ? hl : hh);
  }
  __syncthreads();
}

// First top-p level: a monotone, log-scale bin of a weight.  q < 64 has a
// bin of its own; larger q falls in bin 32 + 32 (e - 5) + m, e its highest
// set bit and m the 5 bits below, a bin of width 2^(e - 5).
__device__ __forceinline__ int sp_qbin(uint64_t q) {
  if (q < 64) return (int)q;
  const int e = 63 - __clzll((long long)q);
  return 32 + 32 * (e - 5) + (int)((q >> (e - 5)) & 31);
}
// the same from the weight before the floor (which moves no bit that it reads)
__device__ __forceinline__ int sp_fbin(float f) {
  return f < 64.f ? (int)f : (int)(__float_as_uint(f) >> 18) - (32 * (127 + 5) - 32);
}
// lowest weight of bin b and the number of its free low bits
__device__ __forceinline__ void sp_qbin_range(int b, uint64_t &lo, int &bits) {
  if (b < 64) {
    lo = (uint64_t)b;
    bits = 0;
  } else {
    const int e = 5 + (b - 32) / 32, m = (b - 32) % 32;
    bits = e - 5;
    lo = (uint64_t)(32 + m) << bits;
  }
}

// hist[0] = total - hist[1..nb) (bin 0 was not accumulated)
__device__ void sp_fill_bin0(SampleLds &S, int nb, uint64_t total) {
  uint64_t v = 0;
  for (int b = 1 + (int)threadIdx.x; b < nb; b += SP_T) v += S.hist[b];
  uint64_t sum;
  sp_scan(v, S.red, sum);
  if (threadIdx.x == 0) S.hist[0] = total - sum;
  __syncthreads();
}

__device__ __forceinline__ void sp_clear(SampleLds &S, int nb) {
  for (int b = threadIdx.x; b < nb; b += SP_T) S.hist[b] = 0;
}

// wave-aggregated append: the slot of this lane's element when pred holds
__device__ __forceinline__ int sp_append(bool pred, int *counter) {
  const uint64_t mask = __ballot(pred);
  if (!mask) return -1;
  const int lane = threadIdx.x & 63, leader = __ffsll((unsigned long long)mask) - 1;
  int base = 0;
  if (lane == leader) base = atomicAdd(counter, __popcll(mask));
  base = __shfl(base, leader, 64);
  return pred ? base + __popcll(mask & ((1ull << lane) - 1ull)) : -1;
}

// smallest of the threads' v, in every thread
__device__ uint32_t sp_min(uint32_t v, uint32_t (&red)[ROW_W]) {
  v = wave_min_u32(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return wave_min_u32(red[threadIdx.x & (ROW_W - 1)]);
}

__device__ __forceinline__ float at4(const float4 &v, int e) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; }

// f(index, logit, valid) for every element
template <typename F>
__device__ __forceinline__ void sp_row(const RowPart &R, F f) {
  row_walk(
      R,
      [&](int c, const float4 &v, auto n) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f(c + e, at4(v, e), e < n);
      },
      [](int) {});
}

// The weights of the row's candidates (order key at least kmin; FILT: kmin is
// not 0): f(index, weight before the floor, weight) for each, and per piece the
// sum of what f returns, into S.pm when PIECES.
template <bool FILT, bool PIECES, typename F>
__device__ __forceinline__ void sp_weights(SampleLds &S, const RowPart &R, int V, uint32_t kmin, float mx, float inv_t,
                                           F f) {
  uint64_t acc = 0;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int per = (row_chunk(V) + SP_PIECE - 1) / SP_PIECE;  // pieces a wave
  row_walk(
      R,
      [&](int c, const float4 &v, auto n) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float l = at4(v, e);
          const bool cand = e < n && (!FILT || order_key(l) >= kmin);
          const float w40 = cand ? f_weight(l, mx, inv_t) : 0.f;
          acc += f(c + e, w40, (uint64_t)w40);
        }
      },
      [&](int batch) {
        if constexpr (PIECES) {
          acc = wave_scan(acc);
          if (lane == 63) S.pm[w * per + batch] = acc;
          acc = 0;
        }
      });
}

// Piece of element c, for the masses of S.pm.
__device__ __forceinline__ int sp_piece(int V, int c) {
  const int chunk = row_chunk(V), per = (chunk + SP_PIECE - 1) / SP_PIECE;
  return c / chunk * per + c % chunk / SP_PIECE;
}

// Top-p threshold among n <= SP_SMALL listed weights with `above` mass over
// all of them: S.sel[0] = the largest whose heavier-or-equal weights reach
// need, S.sel[2] = that mass.
__device__ void sp_reach(SampleLds &S, const uint64_t *list, int n, uint64_t above, uint64_t need) {
  const int tid = threadIdx.x;
  const uint64_t q = tid < n ? list[tid] : 0;
  uint64_t mass = above;
  if (tid < n)
    for (int j = 0; j < n; ++j) {
      const uint64_t o = list[j];
      mass += o >= q ? o : 0;
    }
  const bool reach = tid < n && mass >= need;
  if (tid == 0) S.sel[0] = 0;
  __syncthreads();
  if (reach) atomicMax((unsigned long long *)&S.sel[0], (unsigned long long)q);
  __syncthreads();
  if (reach && q == S.sel[0]) S.sel[2] = mass;
  __syncthreads();
}

__global__ __launch_bounds__(SP_T) void sample_kernel(const float *__restrict__ logits, int64_t ld, int V,
                                                       const SampleParams *__restrict__ prm, const int32_t *out_slot,
                                                       int32_t *slot_tok, int32_t *tok_out) {
  __shared__ SampleLds S;
  const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const RowPart R = row_part(logits, ld, m, V);
  const SampleParams P = prm[m];
  const bool sampled = P.temperature > 0.f && P.top_p > 0.f && V > 1;
  const bool topk = sampled && P.top_k > 0 && P.top_k < V;
  // 1. the maximum
  const RowBest best = row_best(R);
  const float mx = row_max(best, S.fmax);
  int token = -1;  // none yet: the lowest index among the maxima
  if (sampled) {
    const float inv_t = 1.f / P.temperature;
    uint32_t kmin = 0;
    bool in_lds = false;  // candidates (key >= kmin) listed in cq / ci
    if (topk) {
      // 2. top-k threshold: the top_k-th largest order key
      const uint64_t k = (uint64_t)P.top_k;
      bool listed = false;
      int lev0 = 0;          // first radix level over the list
      uint32_t prefix = 0;   // the threshold's bits above that level
      uint64_t above = 0;    // elements above the prefix
      if (tid == 0) S.n_list = 0;
      if (!__syncthreads_or(best.nan) && P.top_k <= SP_FASTK) {
        // L: bins of the lanes' maxima, spread over their own range (the bin
        // of a key is monotone in it), hold at least top_k from L's bin up
        const uint32_t kb = order_key(best.v);
        const uint32_t klo = sp_min(kb, S.kred), khi = order_key(mx);
        const float scale = (float)SP_NB / ((float)(khi - klo) + 1.f);
        const int bin = min(SP_NB - 1, (int)((float)(kb - klo) * scale));
        sp_clear(S, SP_NB);
        __syncthreads();
        atomicAdd((unsigned long long *)&S.hist[bin], 1ull);
        __syncthreads();
        sp_select(S, SP_NB, k, 0);
        const uint32_t kl = sp_min(bin >= (int)S.sel[1] ? kb : 0xFFFFFFFFu, S.kred);
        const bool mine = kb >= kl;
        if (__ballot(mine)) {
          row_walk(
              R,
              [&](int c, const float4 &v, auto n) {
                // no lane here reaches L in this piece, most often
                const float m4 = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
                if (!__ballot(mine && order_key(m4) >= kl)) return;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const uint32_t key = order_key(at4(v, e));
                  const int slot = sp_append(mine && e < n && key >= kl, &S.n_list);
                  if (slot >= 0 && slot < SP_CAP) {
                    S.lv[slot] = key;
                    S.li[slot] = c + e;
                  }
                }
              },
              [](int) {});
        }
        __syncthreads();
        listed = S.n_list <= SP_CAP;
      }
      if (!listed) {
        // histograms over the row, in 11 + 11 + 10 bits; the first level's bin
        // and those above it into the list when they fit
        sp_clear(S, SP_NB);
        __syncthreads();
        if (tid == 0) S.n_list = 0;
        sp_row(R, [&](int, float l, bool ok) {
          if (ok) atomicAdd((unsigned long long *)&S.hist[order_key(l) >> 21], 1ull);
        });
        __syncthreads();
        sp_select(S, SP_NB, k, 0);
        const uint32_t b0 = (uint32_t)S.sel[1];
        above = S.sel[0];
        listed = S.sel[2] <= SP_CAP;  // elements in bins >= b0
        lev0 = 1;
        prefix = b0 << 21;
        __syncthreads();
        if (listed) {
          sp_row(R, [&](int c, float l, bool ok) {
            const uint32_t key = order_key(l);
            const int slot = sp_append(ok && (key >> 21) >= b0, &S.n_list);
            if (slot >= 0 && slot < SP_CAP) {
              S.lv[slot] = key;
              S.li[slot] = c;
            }
          });
          __syncthreads();
        }
      }
      const int n = S.n_list;
      if (listed && n <= SP_SMALL) {
        // the key with fewer than top_k above it and at least top_k from it up
        if (tid < n) {
          const uint32_t key = (uint32_t)S.lv[tid];
          int gt = 0, ge = 0;
          for (int j = 0; j < n; ++j) {
            const uint32_t o = (uint32_t)S.lv[j];
            gt += o > key;
            ge += o >= key;
          }
          if (gt < P.top_k && P.top_k <= ge) S.sel[3] = key;
        }
        __syncthreads();
        prefix = (uint32_t)S.sel[3];
      } else {
        for (int level = lev0; level < 3; ++level) {
          const int sh = level == 0 ? 21 : level == 1 ? 10 : 0, nb = level == 2 ? 1024 : SP_NB;
          const uint32_t pmask = level == 0 ? 0u : level == 1 ? 0xFFE00000u : 0xFFFFFC00u;
          sp_clear(S, nb);
          __syncthreads();
          if (listed) {
            for (int j = tid; j < n; j += SP_T) {
              const uint32_t key = (uint32_t)S.lv[j];
              if ((key & pmask) == prefix) atomicAdd((unsigned long long *)&S.hist[(key >> sh) & (nb - 1)], 1ull);
            }
          } else {
            sp_row(R, [&](int, float l, bool ok) {
              const uint32_t key = order_key(l);
              if (ok && (key & pmask) == prefix)
                atomicAdd((unsigned long long *)&S.hist[(key >> sh) & (nb - 1)], 1ull);
            });
          }
          __syncthreads();
          sp_select(S, nb, k, above);
          above = S.sel[0];
          prefix |= (uint32_t)S.sel[1] << sh;
          __syncthreads();
        }
      }
      kmin = prefix;
      // the candidates, when few, into the draw list
      if (listed) {
        if (tid == 0) S.n_cand = 0;
        __syncthreads();
        for (int j0 = 0; j0 < n; j0 += SP_T) {
          const int j = j0 + tid;
          const bool cand = j < n && (uint32_t)S.lv[j] >= kmin;
          const int slot = sp_append(cand, &S.n_cand);
          if (slot >= 0 && slot < SP_DRAW) {
            S.cq[slot] = q_weight(key_float((uint32_t)S.lv[j]), mx, inv_t);
            S.ci[slot] = S.li[j];
          }
        }
        __syncthreads();
        in_lds = S.n_cand <= SP_DRAW;
      }
    }
    // 3. candidate weights: their total, the top-p threshold tmin, the kept
    // mass zk and, for a draw over the row, the kept mass of every piece
    const uint32_t pfix = P.top_p >= 1.f ? (1u << 24) : max(1u, (uint32_t)(P.top_p * 16777216.0f));
    const bool topp = pfix < (1u << 24);
    const int nc = in_lds ? S.n_cand : 0;
    uint64_t tmin = 0, zk = 0;
    if (in_lds && nc <= SP_SMALL) {
      const uint64_t q = tid < nc ? S.cq[tid] : 0;
      uint64_t z;
      sp_scan(q, S.red, z);
      zk = z;
      if (topp) {
        sp_reach(S, S.cq, nc, 0, mul_shift24(z, pfix, true));
        tmin = S.sel[0];
        zk = S.sel[2];
      }
    } else if (!topp) {
      if (in_lds) {
        sp_scan(tid < nc ? S.cq[tid] : 0, S.red, zk);
      } else {
        S.pm[tid] = 0;
        __syncthreads();
        auto all = [](int, float, uint64_t q) { return q; };
        if (kmin) sp_weights<true, true>(S, R, V, kmin, mx, inv_t, all);
        else sp_weights<false, true>(S, R, V, 0, mx, inv_t, all);
        __syncthreads();
        sp_scan(S.pm[tid], S.red, zk);
      }
    } else {
      uint64_t z = 0;
      sp_clear(S, SP_NB);
      __syncthreads();
      // bin 0 is left out and later set to the total minus the other bins
      if (in_lds) {
        if (tid < nc) {
          z = S.cq[tid];
          if (z) atomicAdd((unsigned long long *)&S.hist[sp_qbin(z)], (unsigned long long)z);
        }
      } else {
        // The threshold cannot lie below a weight Q0 with V Q0 <= Z - need (what
        // is lighter then weighs less than what need leaves out), and Z is at
        // least the sum over the lanes' maxima: bins below Q0's are not
        // counted, which spares most rows half of the atomics.
        uint64_t zlow;
        sp_scan(order_key(best.v) >= kmin ? q_weight(best.v, mx, inv_t) : 0, S.red, zlow);
        const uint64_t spare = mul_shift24(zlow, (1u << 24) - pfix, false);
        uint64_t q0;
        int q0_bits;
        sp_qbin_range(sp_qbin(spare > 2 ? (spare - 2) / (uint32_t)V : 0), q0, q0_bits);
        const float q0f = fmaxf(1.f, (float)q0);  // six significant bits: exact
        auto bins = [&](int, float w40, uint64_t q) {
          if (w40 >= q0f) atomicAdd((unsigned long long *)&S.hist[sp_fbin(w40)], (unsigned long long)q);
          z += q;
          return (uint64_t)0;
        };
        if (kmin) sp_weights<true, false>(S, R, V, kmin, mx, inv_t, bins);
        else sp_weights<false, false>(S, R, V, 0, mx, inv_t, bins);
      }
      uint64_t ztot;
      sp_scan(z, S.red, ztot);
      z = ztot;
      sp_fill_bin0(S, SP_NB, z);
      // a log-scale first level, then the free low bits of the chosen bin, ten
      // at a time
      const uint64_t need = mul_shift24(z, pfix, true);
      sp_select(S, SP_NB, need, 0);
      const int b0 = (int)S.sel[1];
      uint64_t above = S.sel[0];
      zk = S.sel[2];
      __syncthreads();
      uint64_t prefix;
      int rem;
      sp_qbin_range(b0, prefix, rem);
      bool listed = in_lds;
      int n = nc;
      if (!in_lds) {
        // weights above the bin are kept, and those of the bin, which the
        // remaining levels refine, listed (a bin of one weight is kept whole)
        const uint64_t lo = prefix, hi = rem > 0 ? prefix + (1ull << rem) : prefix;
        if (tid == 0) S.n_list = 0;
        S.pm[tid] = 0;
        __syncthreads();
        // compared before the floor: lo and hi are whole, of six bits
        const float lof = fmaxf(1.f, (float)lo), hif = (float)hi;
        auto split = [&](int c, float w40, uint64_t q) {
          const int slot = sp_append(w40 >= lof && w40 < hif, &S.n_list);
          if (slot >= 0 && slot < SP_CAP) {
            S.lv[slot] = q;
            S.li[slot] = c;
          }
          return w40 >= hif ? q : 0;
        };
        if (kmin) sp_weights<true, true>(S, R, V, kmin, mx, inv_t, split);
        else sp_weights<false, true>(S, R, V, 0, mx, inv_t, split);
        __syncthreads();
        n = S.n_list;
        listed = n <= SP_CAP;
      }
      if (!in_lds && listed && rem > 0 && n <= SP_SMALL) {
        sp_reach(S, S.lv, n, above, need);
        prefix = S.sel[0];
        zk = S.sel[2];
        rem = 0;
      }
      while (rem > 0) {
        const int take = min(10, rem), sh = rem - take, nb = 1 << take;
        const uint64_t pmask = ~0ull << rem;
        const uint64_t bucket = zk - above;  // mass of the bin being refined
        sp_clear(S, nb);
        __syncthreads();
        auto refine = [&](uint64_t q) {
          if ((q & pmask) == prefix && ((q >> sh) & (nb - 1)))
            atomicAdd((unsigned long long *)&S.hist[(q >> sh) & (nb - 1)], (unsigned long long)q);
        };
        if (in_lds) {
          if (tid < nc) refine(S.cq[tid]);
        } else if (listed) {
          for (int j = tid; j < n; j += SP_T) refine(S.lv[j]);
        } else {
          sp_weights<true, false>(S, R, V, kmin, mx, inv_t, [&](int, float, uint64_t q) {
            if (q) refine(q);
            return (uint64_t)0;
          });
        }
        __syncthreads();
        sp_fill_bin0(S, nb, bucket);
        sp_select(S, nb, need, above);
        above = S.sel[0];
        prefix |= S.sel[1] << sh;
        zk = S.sel[2];
        rem = sh;
        __syncthreads();
      }
      tmin = prefix;
      if (!in_lds) {
        if (listed) {  // the listed weights that are kept join their pieces
          for (int j = tid; j < n; j += SP_T)
            if (S.lv[j] >= tmin)
              atomicAdd((unsigned long long *)&S.pm[sp_piece(V, S.li[j])], (unsigned long long)S.lv[j]);
        } else {
          sp_weights<true, true>(S, R, V, kmin, mx, inv_t,
                                 [&](int, float, uint64_t q) { return q >= tmin ? q : (uint64_t)0; });
        }
        __syncthreads();
      }
    }
    // 4. draw: r in [0, zk), the kept candidate (q >= tmin) whose cumulative
    // interval in vocabulary order holds r
    uint32_t c4[4] = {P.counter[0], P.counter[1], P.counter[2], 0x53414D50u};
    philox4x32_10(c4, P.key[0], P.key[1]);
    const uint64_t r = mul_shift24(zk, c4[0] >> 8, false);
    if (tid == 0) S.found = -1;
    __syncthreads();
    if (in_lds) {
      if (tid < nc) {
        const uint64_t q = S.cq[tid];
        const int i = S.ci[tid];
        if (q >= tmin) {
          uint64_t pre = 0;
          for (int j = 0; j < nc; ++j) {
            const uint64_t qj = S.cq[j];
            if (qj >= tmin && S.ci[j] < i) pre += qj;
          }
          if (r >= pre && r < pre + q) S.found = i;
        }
      }
    } else {
      // the piece that holds r, then the element in it: four a thread
      const uint64_t run = S.pm[tid];
      uint64_t tot;
      uint64_t pre = sp_scan(run, S.red, tot) - run;
      if (tid == 0) S.pick = -1;
      __syncthreads();
      if (run > 0 && r >= pre && r < pre + run) {
        S.pick = tid;
        S.sel[3] = pre;
      }
      __syncthreads();
      const int p = S.pick;
      if (p >= 0) {
        const int chunk = row_chunk(V), per = (chunk + SP_PIECE - 1) / SP_PIECE;
        const int end = min(V, (p / per + 1) * chunk);
        const int c = p / per * chunk + p % per * SP_PIECE + tid * 4;
        uint64_t q4[4], loc = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          q4[e] = 0;
          if (tid < SP_PIECE / 4 && c + e < end) {
            const float l = R.row[c + e];
            if (order_key(l) >= kmin) {
              const uint64_t q = q_weight(l, mx, inv_t);
              if (q >= tmin) q4[e] = q;
            }
          }
          loc += q4[e];
        }
        uint64_t pl = S.sel[3] + sp_scan(loc, S.red, tot) - loc;
        if (loc > 0 && r >= pl && r < pl + loc) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (q4[e] && r >= pl && r < pl + q4[e]) S.found = c + e;
            pl += q4[e];
          }
        }
      }
    }
    __syncthreads();
    token = S.found;
  }
  if (token < 0) token = row_first(R, best, mx, S.imax);
  if (tid == 0) {
    if (out_slot) slot_tok[out_slot[m]] = token;
    tok_out[m] = token;
  }
}

void launch_sample(const float *logits, int64_t ld, int M, int V, const SampleParams *prm, const int32_t *out_slot,
                   int32_t *slot_tok, int32_t *tok_out, hipStream_t s) {
  if (M <= 0) return;
  sample_kernel<<<M, SP_T, 0, s>>>(logits, ld, V, prm, out_slot, slot_tok, tok_out);
}

template <typename T>
__global__ void init_weight_kernel(T *dst, uint32_t k0, uint32_t k1, uint32_t tid, int64_t rows,
                                   int64_t cols, float stdv, int perm, int hd, bool bf16_values, bool packed,
                                   int64_t row0, int64_t fused_ns) {
  const int64_t n = rows * cols;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    uint32_t c[4] = {(uint32_t)e, (uint32_t)((uint64_t)e >> 32), tid, 0u};
    philox4x32_10(c, k0, k1);
    int s = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += (c[w] & 1023u) + ((c[w] >> 10) & 1023u) + ((c[w] >> 20) & 1023u);
    float v = ((float)(s - 6138) * stdv) * 0x1p-10f;
    if (bf16_values) v = bf16_to_f32(f32_to_bf16(v));
    const int64_t r = e / cols, col = e % cols;
    int64_t dr = r;
    if (perm == PERM_ROPE) {
      const int64_t h = r / hd, i = r % hd;
      dr = h * hd + (i < hd / 2 ? 2 * i : 2 * (i - hd / 2) + 1);
    } else if (perm == PERM_GATE) {
      dr = 2 * r;
    } else if (perm == PERM_UP) {
      dr = 2 * r + 1;
    }
    dst[packed ? wpack_off(row0 + dr, col, fused_ns) : dr * cols + col] = Act<T>::st(v);
  }
}

template <typename T>
void launch_init_weight(T *dst, uint32_t k0, uint32_t k1, uint32_t tensor_id, int64_t rows,
                        int64_t cols, float stdv, int perm, int head_dim, bool bf16_values, bool packed,
                        int64_t row0, int64_t fused_rows, hipStream_t s) {
  const int64_t n = rows * cols;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
  init_weight_kernel<T><<<(unsigned)blocks, 256, 0, s>>>(dst, k0, k1, tensor_id, rows, cols, stdv, perm,
                                                        head_dim, bf16_values, packed, row0,
                                                        wpack_ns(fused_rows));
}

__global__ void fill_f32_kernel(float *dst, int64_t n, float v) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    dst[e] = v;
}

void launch_fill_f32(float *dst, int64_t n, float v, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
  if (n > 0) fill_f32_kernel<<<(unsigned)blocks, 256, 0, s>>>(dst, n, v);
}

#define INST(T)                                                                                   \
  template void launch_embed<T>(const T *, const int32_t *, const int32_t *, const int32_t *,     \
                                const int32_t *, float *, int, int, int, hipStream_t);            \
  template void launch_rmsnorm<T>(float *, const float *, int, int64_t, const int32_t *,          \
                                  const float *, T *, int, int, float, hipStream_t);              \
  template void launch_init_weight<T>(T *, uint32_t, uint32_t, uint32_t, int64_t, int64_t, float, \
                                      int, int, bool, bool, int64_t, int64_t, hipStream_t);
INST(float)
INST(bf16_t)
INST(f16_t)
#undef INST

}  // namespace lp
