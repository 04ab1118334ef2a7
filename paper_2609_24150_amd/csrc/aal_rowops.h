// Workgroup-per-row building blocks shared by the streaming kernels.
#pragma once

#include "aal_device.h"

#include <limits.h>

namespace aal {

constexpr int kRowBlock = 256;
constexpr int kRowWaves = kRowBlock / kWave;
// Threads per workgroup and vectors per thread and round of a row pass.
template <int B, int N>
struct RowShape {
  static constexpr int kBlock = B;
  static constexpr int kU = N;
};

static inline int row_vectors(int V, int vec) { return V / vec + (V % vec != 0); }

// The shape of a pass that reduces one row per workgroup: calls f with it.
// A thread works through all U vectors of a round, the absent ones too, so a
// short row takes the shape that its vectors just fill; one workgroup per CU is
// left with few long rows, which then take as many threads as the CU holds of
// them.  UL: U of the other rows, 4, or 2 for the GRPO pass, which reads three
// arrays.  Kernel times against 256 x UL, us:
//   up to 64 vectors    14,336 x 500 bf16: WTV 51.2 -> 10.9, slice partials
//                       42.7 (ragged) -> 8.2; 512 x 500 WTV 5.0 -> 3.4
//   up to 512           WTV 14,336 x 1,000 66.7 -> 16.9, x 2,000 97.3 -> 34.2; up
//                       to 1,024 rows more threads of fewer vectors: 768 x 1,003
//                       10.9 -> 5.5 (6.5 with 64 x 2), 512 x 2,000 6.9 -> 4.7,
//                       512 x 4,000 7.3 -> 5.8
//   few rows, over 1,024 vectors: 512 x 16,000 15.0 -> 13.6, 256 x 128,256
//                       53.3 -> 39.3; 768 x 16,000 is slower that way (16.6 ->
//                       17.8), as is the GRPO pass above 256 rows (320 x 128,256
//                       fp32 83 -> 94)
template <int UL, class F>
static inline void with_row_shape(int64_t rows, int V, int vec, F&& f) {
  const int ng = row_vectors(V, vec);
  if (ng <= 64) return f(RowShape<64, 1>{});
  if (ng <= 512) {
    if (rows > 1024) return f(RowShape<64, 2>{});
    return ng <= 128 ? f(RowShape<128, 1>{}) : ng <= 256 ? f(RowShape<256, 1>{}) : f(RowShape<256, 2>{});
  }
  if (ng > 1024 && rows <= (UL == 4 ? 512 : 256))
    return rows <= 256 && ng > (UL == 4 ? 2048 : 4096) ? f(RowShape<1024, 2>{}) : f(RowShape<512, 2>{});
  f(RowShape<kRowBlock, UL>{});
}

// U of a pass without a reduction (the gradient passes, 256 threads), called
// with it: one vector per thread where those cover the row (WTV over 512 rows
// of 1,003 bf16 3.8 -> 3.6 us, 14,336 rows 21.4 -> 17.1).
template <class F>
static inline void with_grad_shape(int V, int vec, F&& f) {
  row_vectors(V, vec) <= kRowBlock ? f(RowShape<kRowBlock, 1>{}) : f(RowShape<kRowBlock, 4>{});
}

// Workgroups per row of such a pass: as many as bring the launch to 2048
// workgroups of 256 threads, eight per CU, each with at least one round of U
// vectors per thread.
static inline unsigned row_splits(int64_t rows, int V, int vec, int U) {
  const int64_t rounds = (int64_t(V) / vec + kRowBlock * U - 1) / (kRowBlock * U);
  const int64_t want = (2048 + rows - 1) / rows;
  return unsigned(want < rounds ? want : rounds > 0 ? rounds : 1);
}

// The 16-byte vectors that cover one row of V elements.  ALIGNED: V is a
// multiple of the vector, so every row is whole vectors.  Otherwise a row
// starts `head` elements past a vector boundary (all logit and gradient arrays
// are 16-byte aligned and share the element index, so a row has the same
// phase in each of them): its first and last vectors are shared with the
// neighbouring rows and are loaded whole like the others, then the elements
// outside the row become -inf.  Only the array's very last vector may reach
// past the allocation: in its place the array's last 16 bytes are loaded, by
// the same instruction, and moved to where they belong (an array of less than
// 16 bytes is read element by element).  The stores at a row's edges go
// element by element.  Against element-by-element accesses of the whole row:
// the simulation over 447,252 rows of 2,587 bf16 logits 4.12 -> 1.51 ms, the
// KL + TV passes over 768 rows of 50,001 145 + 77 -> 72 + 46 us, the WTV passes
// over 1792 rows of 32,001 117 + 75 -> 78 + 68 us.
typedef u32x4 u32x4_any __attribute__((aligned(2)));  // a vector at any element

template <class TI, bool ALIGNED>
struct RowVecs {
  static constexpr int E = TI::kVec;
  int64_t g0;  // vector index of the row's first vector
  int ng;      // vectors that cover the row
  int nfull;   // of them, those that lie inside the array
  int nload;   // and those that raw() reads: all, unless the array is shorter than a vector
  int last;    // element past g0 * E at which the array's last 16 bytes start
  int head;    // elements of the first vector before the row
  int V;

  // rows (and the splits of a gradient pass) reach a kernel as arguments:
  // gridDim would come with the runtime's hidden ones, 1.3 us more to enqueue a
  // WTV call (13.9 against 15.2 without Python).
  __device__ __forceinline__ RowVecs(int64_t row, int64_t rows, int v) : V(v) {
    if constexpr (ALIGNED) {
      nload = nfull = ng = v / E;
      g0 = row * int64_t(ng);
      head = last = 0;
    } else {
      const int64_t e0 = row * int64_t(v);
      g0 = e0 / E;
      head = int(e0 - g0 * E);
      ng = int((int64_t(head) + v + E - 1) / E);
      const int64_t end = rows * v - g0 * E;  // the array's, from the row's first vector on
      nfull = int(min(int64_t(ng), end / E));
      nload = rows * v >= E ? ng : 0;
      last = int(min(end - E, int64_t(INT_MAX)));
    }
  }
  // index in the row of element e of vector gi (outside [0, V) at the edges)
  __device__ __forceinline__ int index(int gi, int e) const { return gi * E + e - head; }
  __device__ __forceinline__ bool whole(int gi) const {
    return ALIGNED || (index(gi, 0) >= 0 && index(gi, 0) <= V - E);
  }
  // the vector's 16 bytes, or the array's last 16 if it reaches past them
  __device__ __forceinline__ u32x4 raw(const void* base, int gi) const {
    if constexpr (ALIGNED) {
      return __builtin_nontemporal_load(static_cast<const u32x4*>(base) + g0 + gi);
    } else {
      const typename TI::storage* p = static_cast<const typename TI::storage*>(base) + g0 * E;
      return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(p + min(gi * E, last)));
    }
  }
  // An edge vector of which raw() gave w: moved to its place where it is the
  // array's last, and -inf outside the row, by whole words through one bit per
  // element.  Unrolled element loads at every edge site held 120 registers (of
  // the fp32 passes, 164 against 46 for aligned rows); a rolled loop over them,
  // each load waited for, cost small calls a round trip per element (the row
  // pass over 300 rows of 5,003 bf16: 10.0 us against 7.9).
  __device__ __forceinline__ u32x4 edge(const void* base, int gi, u32x4 w) const {
    using T = typename TI::storage;
    constexpr int EPW = E / 4, kBits = 32 / EPW;
    const int i0 = index(gi, 0);
    const int lo = max(0, -i0), hi = min(E, V - i0);  // the row's elements of the vector
    if (gi >= nload) {
#pragma unroll 1
      for (int e = lo; e < hi; ++e) {
        const T x = static_cast<const T*>(base)[(g0 + gi) * E + e];
        const uint32_t b = EPW == 2 ? uint32_t(__builtin_bit_cast(typename TI::bits, x)) << (e % EPW * 16)
                                    : uint32_t(__builtin_bit_cast(typename TI::bits, x));
        const uint32_t keep = e % EPW ? 0xffffu : 0u;  // the word's lower element, written before
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (e / EPW == q) w[q] = (w[q] & keep) | b;
      }
    } else if (gi >= nfull) {
      // w starts at element `last` and the vector at gi * E: down by the difference
      const int by = gi * E - last, words = by / EPW;
#pragma unroll
      for (int k = 2; k > 0; k /= 2)
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = words & k ? (q + k < 4 ? w[q + k] : 0u) : w[q];
      if constexpr (EPW == 2) {
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = __builtin_amdgcn_alignbit(q < 3 ? w[q + 1] : 0u, w[q], by % EPW * kBits);
      }
    }
    const uint32_t in = ((1u << hi) - 1u) & ~((1u << lo) - 1u);
    const u32x4 out = none();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t m = uint32_t(__builtin_amdgcn_sbfe(int32_t(in), q * EPW, 1));
      if constexpr (EPW == 2)
        m = (m & 0xffffu) | (uint32_t(__builtin_amdgcn_sbfe(int32_t(in), q * EPW + 1, 1)) << kBits);
      w[q] = (w[q] & m) | (out[q] & ~m);
    }
    return w;
  }
  static __device__ __forceinline__ u32x4 none() {
    typename TI::storage x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = TI::neg_inf();
    u32x4 w;
    __builtin_memcpy(&w, x, sizeof w);
    return w;
  }
  // vector gi, -inf outside the row
  __device__ __forceinline__ u32x4 load(const void* base, int gi) const {
    u32x4 w = none();
    if (gi < nload) w = raw(base, gi);
    if (!whole(gi) && gi < ng) w = edge(base, gi, w);
    return w;
  }
  // U vectors of each of N arrays, `step` apart from vector `base` on: the
  // loads are issued together, the edges are mended afterwards.
  template <int N, int U>
  __device__ __forceinline__ void load(const void* const (&p)[N], int base, int step, u32x4 (&w)[N][U]) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int gi = base + u * step;
      if (gi < nload) {
#pragma unroll
        for (int n = 0; n < N; ++n) w[n][u] = raw(p[n], gi);
      } else {
#pragma unroll
        for (int n = 0; n < N; ++n) w[n][u] = none();
      }
    }
    if constexpr (!ALIGNED) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int gi = base + u * step;
        if (!whole(gi) && gi < ng) {
#pragma unroll
          for (int n = 0; n < N; ++n) w[n][u] = edge(p[n], gi, w[n][u]);
        }
      }
    }
  }
  template <int U>
  static __device__ __forceinline__ void unpack(const u32x4 (&w)[U], float (&x)[U][E]) {
#pragma unroll
    for (int u = 0; u < U; ++u) TI::unpack(to_uint4(w[u]), x[u]);
  }
  template <class TG>
  __device__ __forceinline__ void store(void* base, int gi, const float (&g)[E]) const {
    if (whole(gi)) {
      store_vec<TG, E>(base, (g0 + gi) * E, g);
      return;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = index(gi, e);
      if (i >= 0 && i < V) TG::store1(base, (g0 + gi) * E + e, g[e]);
    }
  }
};

// Sum of N values (a power of two) in pairs.  The sums of a chunk of a row go
// this way because a thread adds up whole vectors, 16 or 32 values a chunk: one
// after the other they put the acceptances of rows of 2,045 bf16 entries
// 1.26e-7 from 64 bits (root mean square), in pairs 1.01e-7.
template <int N>
static __device__ __forceinline__ float tree_sum(float (&x)[N]) {
#pragma unroll
  for (int h = N / 2; h > 0; h /= 2)
#pragma unroll
    for (int i = 0; i < h; ++i) x[i] += x[i + h];
  return x[0];
}

// Fold a chunk of logits into a lane's running log-sum-exp.
template <int U, int E>
static __device__ __forceinline__ void lse_fold(LseState& st, const float (&x)[U][E], float sc) {
  float m = kNegInf;
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int e = 0; e < E; ++e) m = fmaxf(m, x[u][e]);
  if (!lse_rebase(st, m, sc)) return;
  float s[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = ex2(__builtin_fmaf(x[u][e], sc, -st.msc));
    s[u] = tree_sum(v);
  }
  st.s += tree_sum(s);
}

// The waves' results, one per wave in LDS, are also added in pairs: up to eight
// by every thread, the sixteen of a wide workgroup by the lanes of every wave
// (which for four waves is slower: two lse and two sum reductions per row put
// the WTV call over 14,000 slice rows of 500 bf16 at 118 us against 107).
template <int WAVES>
static __device__ LseState block_lse(LseState st, float sc, LseState* sh) {
  st = wave_lse(st, sc);
  if constexpr (WAVES == 1) return st;
  const int lane = threadIdx.x & (kWave - 1);
  if (lane == 0) sh[threadIdx.x / kWave] = st;
  __syncthreads();
  LseState r;
  if constexpr (WAVES <= 8) {
    float m = sh[0].m;
#pragma unroll
    for (int i = 1; i < WAVES; ++i) m = fmaxf(m, sh[i].m);
    const float msc = m * sc;
    float s[WAVES];
#pragma unroll
    for (int i = 0; i < WAVES; ++i) s[i] = sh[i].s * ex2(sh[i].msc - msc);
    r = m == kNegInf ? lse_init() : LseState{m, msc, tree_sum(s)};
  } else {
    r = wave_lse(lane < WAVES ? sh[lane] : lse_init(), sc);
  }
  __syncthreads();
  return r;
}

template <int WAVES>
static __device__ float block_sum(float v, float* sh) {
  v = wave_sum(v);
  if constexpr (WAVES == 1) return v;
  const int lane = threadIdx.x & (kWave - 1);
  if (lane == 0) sh[threadIdx.x / kWave] = v;
  __syncthreads();
  float r;
  if constexpr (WAVES <= 8) {
    float s[WAVES];
#pragma unroll
    for (int i = 0; i < WAVES; ++i) s[i] = sh[i];
    r = tree_sum(s);
  } else {
    r = wave_sum(lane < WAVES ? sh[lane] : 0.f);
  }
  __syncthreads();
  return r;
}

// Largest value, lowest index among equal values.
template <int WAVES>
static __device__ int block_argmax(float best, int idx, float* shf, int* shi) {
  const float wm = wave_max(best);
  const int wi = wave_min_i(best == wm ? idx : INT_MAX);
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    shf[w] = wm;
    shi[w] = wi;
  }
  __syncthreads();
  float m = shf[0];
  int i = shi[0];
#pragma unroll
  for (int k = 1; k < WAVES; ++k) {
    if (shf[k] > m || (shf[k] == m && shi[k] < i)) {
      m = shf[k];
      i = shi[k];
    }
  }
  __syncthreads();
  return i;
}


}  // namespace aal
