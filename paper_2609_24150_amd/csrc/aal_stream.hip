// Multi-kernel streaming schedule for the EAL and WTV losses.
//
//   k_row_stats   one workgroup per logit row: max / sum-exp of the tempered
//                 draft (and target) logits; EAL: greedy target token and
//                 a = q(x*)  (Eq. acc_greedy); WTV: a second sweep for
//                 a = sum_v min(p, q) and Q< = sum_{q<p} q  (Eq. acc_sample).
//   k_window_scan one thread per window: prefix products P_j, E = sum_k P_k
//                 (Eq. eal_generic), suffix sums S_j and the gradient
//                 coefficient dloss/da_j = -P_j S_j / N  (Eqs. loss_eal, loss_tv).
//   k_loss        deterministic reduction loss = -(1/N) sum_n E_n.
//   k_grad        one workgroup per row: re-streams the logits and writes
//                 dloss/dz_draft through the softmax Jacobian.
//
// This schedule handles every shape; the register-resident schedule is the
// fast path for shapes it supports.
#include "aal_device.h"
#include "aal_internal.h"
#include "aal_rowops.h"

#include <limits.h>

namespace aal {
namespace {

constexpr int kBlock = kRowBlock;
constexpr int kWaves = kRowWaves;

template <class TI, int MODE, bool VEC, int U, int BLK>
__global__ __launch_bounds__(BLK) void k_row_stats(const void* __restrict__ zd, const void* __restrict__ zt,
                                                   int64_t rows, int V, float scd, float sct,
                                                   RowStats* __restrict__ stats) {
  using Rv = RowVecs<TI, VEC>;
  constexpr int E = Rv::E;
  __shared__ LseState sh_lse[BLK / kWave];
  __shared__ float sh_f[BLK / kWave];
  __shared__ int sh_i[BLK / kWave];

  const int64_t row = blockIdx.x;
  const Rv rv(row, rows, V);
  const int64_t e0 = row * int64_t(V);

  LseState sd = lse_init(), st = lse_init();
  float best = kNegInf;
  int bidx = INT_MAX;

  for (int base = threadIdx.x; base < rv.ng; base += BLK * U) {
    u32x4 w[2][U];
    float xd[U][E], xt[U][E];
    rv.load({zd, zt}, base, BLK, w);
    rv.unpack(w[0], xd);
    rv.unpack(w[1], xt);
    lse_fold(sd, xd, scd);
    if constexpr (MODE == int(Mode::kWtv)) {
      lse_fold(st, xt, sct);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < E; ++e)
          if (xt[u][e] > best) {
            best = xt[u][e];
            bidx = rv.index(base + u * BLK, e);
          }
    }
  }

  sd = block_lse<BLK / kWave>(sd, scd, sh_lse);
  const float l2sd = __log2f(sd.s);
  RowStats out;
  out.msc_d = sd.msc;
  out.l2s_d = l2sd;
  out.coef = 0.f;
  if constexpr (MODE == int(Mode::kEal)) {
    int x = block_argmax<BLK / kWave>(best, bidx, sh_f, sh_i);
    if (x == INT_MAX) x = 0;  // a row with no finite target logit: unspecified, stay in bounds
    const float zx = TI::load1(zd, e0 + x);
    out.a = ex2(__builtin_fmaf(zx, scd, -sd.msc) - l2sd);
    out.xstar = x;
    out.msc_t = 0.f;
    out.l2s_t = 0.f;
    out.qlt = 0.f;
  } else {
    st = block_lse<BLK / kWave>(st, sct, sh_lse);
    const float l2st = __log2f(st.s);
    float smin = 0.f, qlt = 0.f;
    for (int base = threadIdx.x; base < rv.ng; base += BLK * U) {
      u32x4 w[2][U];
      float xd[U][E], xt[U][E];
      rv.load({zd, zt}, base, BLK, w);
      rv.unpack(w[0], xd);
      rv.unpack(w[1], xt);
      float am[U], aq[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float vm[E], vq[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const float ld = __builtin_fmaf(xd[u][e], scd, -sd.msc) - l2sd;
          const float lt = __builtin_fmaf(xt[u][e], sct, -st.msc) - l2st;
          const float m = ex2(fminf(ld, lt));
          vm[e] = m;
          vq[e] = (ld < lt) ? m : 0.f;
        }
        am[u] = tree_sum(vm);
        aq[u] = tree_sum(vq);
      }
      smin += tree_sum(am);
      qlt += tree_sum(aq);
    }
    smin = block_sum<BLK / kWave>(smin, sh_f);
    qlt = block_sum<BLK / kWave>(qlt, sh_f);
    out.a = smin;
    out.qlt = qlt;
    out.msc_t = st.msc;
    out.l2s_t = l2st;
    out.xstar = -1;
  }
  if (threadIdx.x == 0) stats[row] = out;
}

// One thread per window.  P_j = prod_{i<j} a_i, E = sum_{k=1..K} P_k,
// S_{K-1} = 1, S_j = 1 + a_{j+1} S_{j+1};  dE/da_j = P_j S_j.
__global__ __launch_bounds__(kBlock) void k_window_scan(RowStats* __restrict__ stats, int64_t N, int K, int mode,
                                                        float inv_t_d, const float* __restrict__ grad_scale,
                                                        float* __restrict__ window_e, float* __restrict__ accept,
                                                        int32_t* __restrict__ xstar) {
  const int64_t n = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (n >= N) return;
  RowStats* s = stats + n * K;
  double P[64];
  double p = 1.0, E = 0.0;
  for (int j = 0; j < K; ++j) {
    P[j] = p;
    p *= double(s[j].a);
    E += p;
  }
  const double scale = grad_scale ? double(*grad_scale) : 1.0;
  const double inv_n = 1.0 / double(N);
  double S = 1.0;
  for (int j = K - 1; j >= 0; --j) {
    const float a = s[j].a;
    const double g = -P[j] * S * inv_n;  // dloss/da_j
    const double factor = (mode == int(Mode::kEal)) ? double(a) * double(inv_t_d) : double(inv_t_d);
    s[j].coef = float(g * scale * factor);
    if (accept) accept[n * K + j] = a;
    if (xstar) xstar[n * K + j] = s[j].xstar;
    S = 1.0 + double(a) * S;
  }
  window_e[n] = float(E);
}

// err (may be null): a resident kernel's error word; set, the loss is NaN (a
// poll timed out and the per-window values are incomplete).
__global__ __launch_bounds__(kBlock) void k_loss(const float* __restrict__ window_e, int64_t N,
                                                 float* __restrict__ loss, const unsigned* __restrict__ err) {
  __shared__ double sh[kWaves];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < N; i += kBlock) acc += double(window_e[i]);
  acc = wave_sum_d(acc);
  if ((threadIdx.x & (kWave - 1)) == 0) sh[threadIdx.x / kWave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = sh[0];
    for (int i = 1; i < kWaves; ++i) t += sh[i];
    loss[0] = (err != nullptr && *err != 0u) ? __builtin_nanf("") : float(-t / double(N));
  }
}

template <class TI, class TG, int MODE, bool VEC, int U>
__global__ __launch_bounds__(kBlock) void k_grad(const void* __restrict__ zd, const void* __restrict__ zt, int64_t rows,
                                                 int splits, int V, float scd, float sct,
                                                 const RowStats* __restrict__ stats, void* __restrict__ grad) {
  using Rv = RowVecs<TI, VEC>;
  constexpr int E = Rv::E;
  constexpr int NT = MODE == int(Mode::kEal) ? 1 : 2;  // logit arrays read
  const int64_t row = blockIdx.x;
  const Rv rv(row, rows, V);
  const RowStats s = stats[row];
  const float c = s.coef;
  const float cA = c * (1.f - s.qlt);  // WTV, entries with q < p
  const float cB = -c * s.qlt;         // WTV, the others
  for (int base = blockIdx.y * kBlock * U + threadIdx.x; base < rv.ng; base += splits * kBlock * U) {
    u32x4 w[NT][U];  // loaded together: a launch of few wavefronts waits once per round
    if constexpr (NT == 2)
      rv.load({zd, zt}, base, kBlock, w);
    else
      rv.load({zd}, base, kBlock, w);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int gi = base + u * kBlock;
      if (gi >= rv.ng) break;
      float xd[E], g[E];
      TI::unpack(to_uint4(w[0][u]), xd);
      if constexpr (MODE == int(Mode::kEal)) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const float q = ex2(__builtin_fmaf(xd[e], scd, -s.msc_d) - s.l2s_d);
          const float d = (rv.index(gi, e) == s.xstar) ? 1.f : 0.f;
          g[e] = c * (d - q);
        }
      } else {
        float xt[E];
        TI::unpack(to_uint4(w[NT - 1][u]), xt);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const float ld = __builtin_fmaf(xd[e], scd, -s.msc_d) - s.l2s_d;
          const float lt = __builtin_fmaf(xt[e], sct, -s.msc_t) - s.l2s_t;
          const float q = ex2(ld);
          g[e] = q * ((ld < lt) ? cA : cB);
        }
      }
      rv.template store<TG>(grad, gi, g);
    }
  }
}

template <class TI, class TG, int MODE, bool VEC>
void grad_launch(const LossArgs& a) {
  const int64_t rows = a.N * a.K;
  with_grad_shape(a.V, TI::kVec, [&](auto sh) {
    constexpr int U = decltype(sh)::kU;
    const unsigned splits = row_splits(rows, a.V, TI::kVec, U);
    k_grad<TI, TG, MODE, VEC, U><<<dim3(unsigned(rows), splits), kBlock, 0, a.stream>>>(
        a.zd, a.zt, rows, int(splits), a.V, a.sc_d, a.sc_t, a.ws.stats, a.grad);
  });
}

template <class TI, int MODE, bool VEC>
hipError_t launch_vec(const LossArgs& a) {
  const int64_t rows = a.N * a.K;
  with_row_shape<4>(rows, a.V, TI::kVec, [&](auto sh) {
    using Sh = decltype(sh);
    k_row_stats<TI, MODE, VEC, Sh::kU, Sh::kBlock><<<dim3(unsigned(rows)), Sh::kBlock, 0, a.stream>>>(
        a.zd, a.zt, rows, a.V, a.sc_d, a.sc_t, a.ws.stats);
  });
  const unsigned wblocks = unsigned((a.N + kBlock - 1) / kBlock);
  k_window_scan<<<wblocks, kBlock, 0, a.stream>>>(a.ws.stats, a.N, a.K, MODE, a.inv_t_d, a.grad_scale, a.window_e,
                                                  a.accept, a.xstar);
  k_loss<<<1, kBlock, 0, a.stream>>>(a.window_e, a.N, a.loss, nullptr);
  if (a.grad) {
    if (a.gd == DType::kBf16)
      grad_launch<TI, GBf16, MODE, VEC>(a);
    else
      grad_launch<TI, GF32, MODE, VEC>(a);
  }
  return hipGetLastError();
}

template <class TI, int MODE>
hipError_t launch_typed(const LossArgs& a) {
  return a.V % TI::kVec == 0 ? launch_vec<TI, MODE, true>(a) : launch_vec<TI, MODE, false>(a);
}

}  // namespace

hipError_t launch_loss_reduce(const LossArgs& a, const unsigned* err) {
  k_loss<<<1, kBlock, 0, a.stream>>>(a.window_e, a.N, a.loss, err);
  return hipGetLastError();
}

hipError_t launch_streaming(const LossArgs& a) {
  if (a.in == DType::kBf16) {
    return a.mode == Mode::kEal ? launch_typed<Bf16, int(Mode::kEal)>(a) : launch_typed<Bf16, int(Mode::kWtv)>(a);
  }
  return a.mode == Mode::kEal ? launch_typed<F32, int(Mode::kEal)>(a) : launch_typed<F32, int(Mode::kWtv)>(a);
}

}  // namespace aal
