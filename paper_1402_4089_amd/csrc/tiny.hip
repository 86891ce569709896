// Small problems: a gradient, L leapfrog updates or a whole HMC transition in one launch of one
// workgroup, with X, the residuals and the state in its LDS.
//
// At n = 500, p = 20, K = 3 a gradient is 60,000 multiply-adds and the general path's two
// kernels per update take 4.3 us each, which is what a launch costs, not the work: a
// transition of ten updates was 23 launches and 99 us. Here an update is three phases between
// workgroup barriers: a thread per row of X forms the row's logits, softmax and residuals; a
// thread per gradient element and row group sums x r over its rows in float64; a thread per
// element adds the prior and applies the kicks and the drift. Latency bounds it (about 3 us per
// update: the float64 exponentials and the serial sums), so it is used while a thread has few
// rows and terms (tiny_fits).
//
// A row's logits are formed in the order of the row-tile kernel's matrix instructions (blocks of
// 16 columns, in a block columns t, 4 + t, 8 + t, 12 + t for t = 0 .. 3, the blocks' sums added in
// turn) and its softmax with the same functions and tree, so log K does not depend on which
// of the two runs but for the order of the float64 sum over rows; the gradient's row sums are
// float64 here where that kernel adds 16 rows at a time in the state's precision.
#include <math.h>

#include "device_common.h"

namespace hmcx {
namespace {

using namespace dev;

constexpr size_t kTinyLds = 150 * 1024;

// LDS sections of a problem, in bytes from the start (each 16-byte aligned).
struct TinyLayout {
  size_t x, b, pos, mom, grad, res, red, total;
  int pitch;                                       // elements between rows of X, odd
};
__host__ __device__ inline TinyLayout tiny_layout(int n, int p, int K, int kp, int threads, size_t ts) {
  TinyLayout l;
  const auto up = [](size_t v) { return (v + 15) / 16 * 16; };
  const size_t pk = (size_t)p * K;
  l.pitch = p | 1;
  l.x = 0;
  l.b = up(l.x + (size_t)n * l.pitch * ts);
  l.pos = up(l.b + (size_t)p * kp * ts);
  l.mom = up(l.pos + pk * ts);
  l.grad = up(l.mom + pk * ts);
  l.res = up(l.grad + pk * ts);
  l.red = up(l.res + (size_t)n * K * ts);
  l.total = up(l.red + (pk > (size_t)threads ? pk : (size_t)threads) * 8);
  return l;
}
int class_pad(int K) { return K == 1 ? 1 : K <= 4 ? 4 : K <= 8 ? 8 : 16; }
int tiny_threads(int64_t n) { return n <= 512 ? 512 : 1024; }

// Sum over the workgroup in a fixed order, the same in every thread.
template <int TH> __device__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < TH / 64; ++w) s += sh[w];
  return s;
}

// Sum of KP values in the order of a 16-lane DPP reduction (pairs, quads, halves).
template <typename T, int KP> __device__ __forceinline__ T tree(const T (&e)[KP]) {
  if constexpr (KP == 1) return e[0];
  T v[KP];
#pragma unroll
  for (int k = 0; k < KP; ++k) v[k] = e[k];
#pragma unroll
  for (int h = 1; h < KP; h *= 2)
#pragma unroll
    for (int k = 0; k < KP; k += 2 * h) v[k] += v[k + h];
  return v[0];
}

template <typename T, int KP, int TH>
__global__ __launch_bounds__(TH) void tiny_kernel(TinyArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double sh[TH / 64];
  const int tid = threadIdx.x;
  const int n = (int)a.n, p = a.p, K = a.K, pk = p * K;
  const TinyLayout l = tiny_layout(n, p, K, KP, TH, sizeof(T));
  T* xs = reinterpret_cast<T*>(smem + l.x);            // [n][pitch]
  T* bs = reinterpret_cast<T*>(smem + l.b);            // [p][KP] position, zero past the free classes
  T* pos = reinterpret_cast<T*>(smem + l.pos);         // [p][K]
  T* mom = reinterpret_cast<T*>(smem + l.mom);
  T* grad = reinterpret_cast<T*>(smem + l.grad);
  T* res = reinterpret_cast<T*>(smem + l.res);         // [n][K]
  double* red = reinterpret_cast<double*>(smem + l.red);
  const T* X = static_cast<const T*>(a.X);
  T* B = static_cast<T*>(a.B);
  T* G = static_cast<T*>(a.G);
  T* eta = static_cast<T*>(a.eta);
  const T h = (T)a.h, eps = (T)a.eps;
  auto pinned = [&](int e) { return a.pin && e % K == K - 1; };
  auto put = [&](int e, T v) {                         // position of element e
    pos[e] = v;
    bs[e / K * KP + e % K] = pinned(e) ? T(0) : v;
  };

  {
    // element tid, tid + TH, .. of the rows, row and column stepped without a division
    const int dr = TH / p, dc = TH - dr * p;
    int r = tid / p, c = tid - r * p;
    while (r < n) {
      T v[8];
      int rr[8], cc[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        rr[u] = r;
        cc[u] = c;
        v[u] = r < n ? X[(int64_t)r * a.ldx + c] : T(0);
        c += dc;
        r += dr + (c >= p);
        c -= c >= p ? p : 0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (rr[u] < n) xs[rr[u] * l.pitch + cc[u]] = v[u];
    }
  }
  for (int i = tid; i < p * KP; i += TH) bs[i] = T(0);
  __syncthreads();

  // start of the trajectory: momentum, opening half kick and drift (equations (hmc1) and the
  // position step)
  const int64_t iter = a.ctr ? a.ctr[0] : a.iter;
  const int64_t t = a.ctr ? a.ctr[0] - a.ctr[1] : a.t;
  const bool rec = t >= 0 && t < a.n_rec;
  double ke0 = 0.0;
  for (int e = tid; e < pk; e += TH) {
    T bt = B[e];
    if (a.mode != 0) {
      T ev;
      if (a.mode == 1) {
        ev = eta[e];
      } else {
        const double xi = a.draw == 1 && rec ? a.normals[t * pk + e] : philox_normal(a.seed, a.chain, iter, e);
        ev = pinned(e) ? T(0) : (T)xi;
        ke0 += 0.5 * (double)ev * (double)ev;
      }
      ev = ev + h * G[e];
      bt = pinned(e) ? T(0) : bt + eps * ev;
      mom[e] = ev;
    }
    put(e, bt);
  }
  __syncthreads();

  // elements of the gradient and row groups: threads e + pk q sum rows q, q + ngrp, ..
  const int ngrp = pk < TH ? TH / pk : 1;
  double logk = 0.0, ke1 = 0.0;
  const int steps = a.mode == 0 ? 1 : a.L;
  for (int st = 1; st <= steps; ++st) {
    double lacc = 0.0;
    for (int i = tid; i < n; i += TH) {
      const T* x = xs + i * l.pitch;
      T z[KP];
      for (int b0 = 0; b0 < p; b0 += 16) {
        T zb[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) zb[k] = T(0);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int j = b0 + 4 * (q & 3) + (q >> 2);
          if (j < p) {
            const T xv = x[j];
#pragma unroll
            for (int k = 0; k < KP; ++k) zb[k] = fma(xv, bs[j * KP + k], zb[k]);
          }
        }
#pragma unroll
        for (int k = 0; k < KP; ++k) z[k] = b0 == 0 ? zb[k] : z[k] + zb[k];
      }
      const int yi = a.y[i];
      if constexpr (KP == 1) {
        if (a.link == 1) {
          const T mu = dev_exp(z[0]);
          res[i] = T(yi) - mu;
          lacc += (double)yi * (double)z[0] - (double)mu;
        } else {
          const T s = yi == 1 ? T(1) : T(-1);
          T ratio;
          double lp;
          probit_row(s * z[0], ratio, lp);
          res[i] = s * ratio;
          lacc += lp;
        }
      } else {
        T mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < KP; ++k)
          if (k < K) mx = fmax(mx, z[k]);
        T ex[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) ex[k] = k < K ? dev_exp(z[k] - mx) : T(0);
        const T se = tree<T, KP>(ex);
        const T inv = dev_rcp(se), lse_shift = dev_log(se);
#pragma unroll
        for (int k = 0; k < KP; ++k) {
          if (k < K) res[i * K + k] = (k == yi ? T(1) : T(0)) - ex[k] * inv;
          lacc += k == yi ? (double)((z[k] - mx) - lse_shift) : 0.0;
        }
      }
    }
    __syncthreads();
    for (int e = tid; e < pk * ngrp; e += TH) {
      const int el = e % pk, j = el / K, k = el % K;
      double s[4] = {0.0, 0.0, 0.0, 0.0};
      int i = e / pk;
      for (; i + 3 * ngrp < n; i += 4 * ngrp) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          s[u] = fma((double)xs[(i + u * ngrp) * l.pitch + j], (double)res[(i + u * ngrp) * K + k], s[u]);
      }
      for (; i < n; i += ngrp) s[0] = fma((double)xs[i * l.pitch + j], (double)res[i * K + k], s[0]);
      red[e] = ((s[0] + s[1]) + s[2]) + s[3];
    }
    __syncthreads();
    const bool last = st == steps;
    double pr = 0.0;
    for (int e = tid; e < pk; e += TH) {
      double gsum = red[e];
      for (int q = 1; q < ngrp; ++q) gsum += red[q * pk + e];
      const bool pin = pinned(e);
      const T bt = pos[e];
      const double b = (double)bt;
      const T gt = pin ? T(0) : (T)(gsum + prior_grad(b, a.prior, a.scale));
      if (last) {
        grad[e] = gt;
        pr += pin ? 0.0 : prior_logd(b, a.prior, a.scale);
      }
      if (a.mode != 0) {
        T ev = mom[e] + h * gt;                        // closing half kick, equation (hmc3)
        if (last) {
          ke1 += 0.5 * (double)ev * (double)ev;
        } else {
          ev = ev + h * gt;                            // opening half kick of the next update
          put(e, pin ? T(0) : bt + eps * ev);          // full position step
        }
        mom[e] = ev;
      }
    }
    if (last) logk = block_sum<TH>(lacc + pr, sh);
    __syncthreads();
  }

  if (a.mode == 0) {
    for (int e = tid; e < pk; e += TH) G[e] = grad[e];
    if (tid == 0) *a.logpost = logk;
    return;
  }
  if (a.mode == 1) {
    for (int e = tid; e < pk; e += TH) {
      B[e] = pos[e];
      eta[e] = mom[e];
      G[e] = grad[e];
    }
    if (tid == 0) *a.logpost = logk;
    return;
  }
  // Metropolis test, selection and records
  ke0 = block_sum<TH>(ke0, sh);
  ke1 = block_sum<TH>(ke1, sh);
  const double logk0 = *a.logpost;
  const double H0 = -logk0 + ke0, H1 = -logk + ke1;
  const double u = a.replay_u && rec ? a.replay_u[t] : philox_uniform(a.seed, a.chain, iter);
  const double it = a.inv_temp && rec ? a.inv_temp[t] : 1.0;
  const bool finite = isfinite(H1);
  const bool acc = finite && (log(u) < (H0 - H1) * it);
  __syncthreads();                                     // every thread has read log K and the counter
  for (int e = tid; e < pk; e += TH) {
    T bnew;
    if (acc) {
      bnew = pos[e];
      B[e] = bnew;
      G[e] = grad[e];
    } else {
      bnew = B[e];
    }
    if (a.sample && rec) static_cast<T*>(a.sample)[t * pk + e] = bnew;
  }
  if (tid == 0) {
    *a.logpost = acc ? logk : logk0;
    if (rec) {
      if (a.accepted) a.accepted[t] = acc ? 1 : 0;
      if (a.divergent) a.divergent[t] = !finite || H1 - H0 > 1000.0 ? 1 : 0;
      if (a.H) { a.H[2 * t] = H0; a.H[2 * t + 1] = H1; }
    }
    if (a.ctr) a.ctr[0] = iter + 1;
  }
}

template <typename T, int KP, int TH>
hipError_t launch_one(const TinyArgs& a, size_t lds, hipStream_t s) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tiny_kernel<T, KP, TH>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((tiny_kernel<T, KP, TH>), dim3(1), dim3(TH), lds, s, a);
  return hipGetLastError();
}

}  // namespace

bool tiny_fits(int64_t n, int64_t p, int K, bool f64) {
  if (n > 1024 || p > 256 || K > 16 || n * p * K > (int64_t)1 << 16) return false;
  return tiny_layout((int)n, (int)p, K, class_pad(K), tiny_threads(n), f64 ? 8 : 4).total <= kTinyLds;
}

template <typename T>
hipError_t launch_tiny(const TinyArgs& a, hipStream_t s) {
  const int kp = class_pad(a.K), th = tiny_threads(a.n);
  const size_t lds = tiny_layout((int)a.n, a.p, a.K, kp, th, sizeof(T)).total;
#define HMC_TINY(KP_)                                                                        \
  if (kp == KP_) return th == 512 ? launch_one<T, KP_, 512>(a, lds, s) : launch_one<T, KP_, 1024>(a, lds, s);
  HMC_TINY(1) HMC_TINY(4) HMC_TINY(8) HMC_TINY(16)
#undef HMC_TINY
  return hipErrorInvalidValue;
}

template hipError_t launch_tiny<float>(const TinyArgs&, hipStream_t);
template hipError_t launch_tiny<double>(const TinyArgs&, hipStream_t);

}  // namespace hmcx
