// Small problems: a gradient, L leapfrog updates or a whole HMC transition in one launch of one
// workgroup, with X, the residuals and the state in its LDS.
//
// At n = 500, p = 20, K = 3 a gradient is 60,000 multiply-adds and the general path's two
// kernels per update take 4.3 us each, which is what a launch costs, not the work: a
// transition of ten updates was 23 launches and 99 us. Here an update is three phases between
// workgroup barriers: a thread per row of X forms the row's logits, softmax and residuals; a
// thread per column of X and group of rows sums x r over its rows in float64 for every free
// class; a thread per element adds the prior and applies the kicks and the drift. LDS reads and
// the latency of the float64 functions bound it, so it is used where its time is below the
// general path's launches (tiny_fits). That transition now takes 45 us, 3.7 per update (timed with
// phases left out: logits 1.3, softmax 1.1, gradient 1.4 of 4.9 in a form with a thread per
// gradient element, whose LDS reads were twice as many), and one gradient 9.6.
//
// A row's logits are formed in the order of the row-tile kernel's matrix instructions (blocks of
// 16 columns, in a block columns t, 4 + t, 8 + t, 12 + t for t = 0 .. 3, the blocks' sums added in
// turn) and its softmax with the same functions and tree, so log K does not depend on which
// of the two runs but for the order of the float64 sum over rows; the gradient's row sums are
// float64 here where that kernel adds 16 rows at a time in the state's precision.
//
// With 1024 threads a lane has 128 registers: in float64, one and eight padded classes keep 68 and
// 92 bytes of scratch per lane.
#include <math.h>

#include "device_common.h"

namespace hmcx {
namespace {

using namespace dev;

constexpr size_t kTinyLds = 150 * 1024;
constexpr int kTinyGroups = 16;                    // row groups of the gradient at most

// LDS sections of a problem, in bytes from the start (each 16-byte aligned). fp: free classes
// (K, or K - 1 with the pinned class) padded to a power of two.
struct TinyLayout {
  size_t x, b, res, red, total;
  int pitch;                                       // elements between rows of X, odd
  int groups;                                      // row groups of the gradient
};
__host__ __device__ inline TinyLayout tiny_layout(int n, int p, int fp, int threads, size_t ts) {
  TinyLayout l;
  const auto up = [](size_t v) { return (v + 15) / 16 * 16; };
  l.pitch = p | 1;
  l.groups = threads / p < kTinyGroups ? threads / p : kTinyGroups;
  l.x = 0;
  l.b = up(l.x + (size_t)n * l.pitch * ts);
  l.res = up(l.b + (size_t)p * fp * ts);
  l.red = up(l.res + (size_t)n * fp * ts);
  l.total = up(l.red + (size_t)l.groups * p * fp * 8);
  return l;
}
int class_pad(int f) { return f <= 1 ? 1 : f <= 2 ? 2 : f <= 4 ? 4 : f <= 8 ? 8 : 16; }
int tiny_threads(int64_t n, int64_t pk) { return n <= 512 && pk <= 512 ? 512 : 1024; }

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

// Sum of N values (a power of two) in the order of a 16-lane DPP reduction.
template <typename T, int N> __device__ __forceinline__ T tree(T (&v)[N]) {
#pragma unroll
  for (int h = 1; h < N; h *= 2)
#pragma unroll
    for (int k = 0; k < N; k += 2 * h) v[k] += v[k + h];
  return v[0];
}

template <typename T, int FP, int TH>
__global__ __launch_bounds__(TH) void tiny_kernel(TinyArgs a) {
  constexpr int KP = 2 * FP < 16 ? 2 * FP : 16;        // padded classes, the pinned one among them
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double sh[TH / 64];
  const int tid = threadIdx.x;
  const int n = (int)a.n, p = a.p, K = a.K, pk = p * K;
  const int F = a.pin ? K - 1 : K;
  const TinyLayout l = tiny_layout(n, p, FP, TH, sizeof(T));
  T* xs = reinterpret_cast<T*>(smem + l.x);            // [n][pitch]
  T* bs = reinterpret_cast<T*>(smem + l.b);            // [p][FP] position, zero past the free classes
  T* res = reinterpret_cast<T*>(smem + l.res);         // [n][FP] residuals of the free classes
  double* red = reinterpret_cast<double*>(smem + l.red);   // [groups][p][FP]
  const T* X = static_cast<const T*>(a.X);
  const T h = (T)a.h, eps = (T)a.eps;

  // this thread's element of the state (row ej, class ek), its row of X and its share of the gradient
  const bool elem = tid < pk;
  const int ej = elem ? tid / K : 0, ek = elem ? tid - ej * K : 0;
  const bool pin = a.pin && ek == K - 1, free = elem && !pin;
  const bool row = tid < n;
  const int gq = tid / p, gj = tid - gq * p;           // gradient: column gj, rows gq, gq + groups, ..
  const int yi = row ? a.y[tid] : 0;
  const T b0 = elem ? static_cast<const T*>(a.B)[tid] : T(0);
  const T g0 = elem && a.mode != 0 ? static_cast<const T*>(a.G)[tid] : T(0);
  {
    // element tid, tid + TH, .. of the rows, row and column stepped without a division
    const int dr = TH / p, dc = TH - dr * p;
    int r = gq, c = gj;
    while (r < n) {
      T v[8];
      int at[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        at[u] = r < n ? r * l.pitch + c : -1;
        v[u] = r < n ? X[(int64_t)r * a.ldx + c] : T(0);
        c += dc;
        r += dr + (c >= p);
        c -= c >= p ? p : 0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (at[u] >= 0) xs[at[u]] = v[u];
    }
  }
  for (int i = tid; i < p * FP; i += TH) bs[i] = T(0);
  for (int i = tid; i < n * FP; i += TH) res[i] = T(0);

  // start of the trajectory: momentum, opening half kick and drift (equations (hmc1) and the
  // position step)
  const int64_t iter = a.ctr ? a.ctr[0] : a.iter;
  const int64_t t = a.ctr ? a.ctr[0] - a.ctr[1] : a.t;
  const bool rec = t >= 0 && t < a.n_rec;
  double ke0 = 0.0, ke1 = 0.0, pr = 0.0, logk = 0.0;
  T pos = b0, mom = T(0), grad = T(0);
  if (elem && a.mode != 0) {
    if (a.mode == 1) {
      mom = static_cast<const T*>(a.eta)[tid];
    } else {
      const double xi = a.draw == 1 && rec ? a.normals[t * pk + tid] : philox_normal(a.seed, a.chain, iter, tid);
      mom = pin ? T(0) : (T)xi;
      ke0 = 0.5 * (double)mom * (double)mom;
    }
    mom = mom + h * g0;
    pos = pin ? T(0) : b0 + eps * mom;
  }
  __syncthreads();
  if (free) bs[ej * FP + ek] = pos;
  // the pinned class's logit: zero, or a NaN in a row that holds an infinity or a NaN
  T zpin = T(0);
  if (row && a.pin)
    for (int j = 0; j < p; ++j) zpin = fma(xs[tid * l.pitch + j], T(0), zpin);
  __syncthreads();

  const int steps = a.mode == 0 ? 1 : a.L;
  for (int st = 1; st <= steps; ++st) {
    double lacc = 0.0;
    if (row) {
      const T* x = xs + tid * l.pitch;
      T z[FP];
      for (int c0 = 0; c0 < p; c0 += 16) {
        T zb[FP];
#pragma unroll
        for (int k = 0; k < FP; ++k) zb[k] = T(0);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int j = c0 + 4 * (q & 3) + (q >> 2);
          if (j < p) {
            const T xv = x[j];
#pragma unroll
            for (int k = 0; k < FP; ++k) zb[k] = fma(xv, bs[j * FP + k], zb[k]);
          }
        }
#pragma unroll
        for (int k = 0; k < FP; ++k) z[k] = c0 == 0 ? zb[k] : z[k] + zb[k];
      }
      bool done = false;
      if constexpr (FP == 1) {
        if (a.link == 1) {
          const T mu = dev_exp(z[0]);
          res[tid] = T(yi) - mu;
          lacc = (double)yi * (double)z[0] - (double)mu;
          done = true;
        } else if (a.link == 2) {
          const T s = yi == 1 ? T(1) : T(-1);
          T ratio;
          probit_row(s * z[0], ratio, lacc);
          res[tid] = s * ratio;
          done = true;
        }
      }
      if (!done) {
        T mx = a.pin ? fmax((T)-INFINITY, zpin) : (T)-INFINITY;
#pragma unroll
        for (int k = 0; k < FP; ++k)
          if (k < F) mx = fmax(mx, z[k]);
        T ex[KP], sum[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) {
          ex[k] = T(0);
          if (k < K) ex[k] = dev_exp((k < FP && k < F ? z[k < FP ? k : 0] : zpin) - mx);
          sum[k] = ex[k];
        }
        const T se = tree<T, KP>(sum);
        const T inv = dev_rcp(se), lse_shift = dev_log(se);
        T zy = zpin;                                   // the label's logit
#pragma unroll
        for (int k = 0; k < FP; ++k)
          if (k < F) {
            res[tid * FP + k] = (k == yi ? T(1) : T(0)) - ex[k] * inv;
            zy = k == yi ? z[k] : zy;
          }
        // as on the row tile: no term for a label outside the 16 padded classes
        if ((unsigned)yi < 16u) lacc = (double)((zy - mx) - lse_shift);
      }
    }
    __syncthreads();
    if (gq < l.groups) {
      double s[FP];
#pragma unroll
      for (int k = 0; k < FP; ++k) s[k] = 0.0;
#pragma unroll 4
      for (int i = gq; i < n; i += l.groups) {
        const double xv = (double)xs[i * l.pitch + gj];
#pragma unroll
        for (int k = 0; k < FP; ++k) s[k] = fma(xv, (double)res[i * FP + k], s[k]);
      }
#pragma unroll
      for (int k = 0; k < FP; ++k) red[(gq * p + gj) * FP + k] = s[k];
    }
    __syncthreads();
    const bool last = st == steps;
    if (elem) {
      double gsum = 0.0;
      if (free) {
#pragma unroll 8
        for (int q = 0; q < l.groups; ++q) gsum += red[(q * p + ej) * FP + ek];
      }
      const double b = (double)pos;
      grad = pin ? T(0) : (T)(gsum + prior_grad(b, a.prior, a.scale));
      if (last) pr = pin ? 0.0 : prior_logd(b, a.prior, a.scale);
      if (a.mode != 0) {
        mom = mom + h * grad;                          // closing half kick, equation (hmc3)
        if (last) {
          ke1 = 0.5 * (double)mom * (double)mom;
        } else {
          mom = mom + h * grad;                        // opening half kick of the next update
          pos = pin ? T(0) : pos + eps * mom;          // full position step
          if (free) bs[ej * FP + ek] = pos;
        }
      }
    }
    if (last) logk = block_sum<TH>(lacc + pr, sh);
    __syncthreads();
  }

  T* B = static_cast<T*>(a.B);
  T* G = static_cast<T*>(a.G);
  if (a.mode != 2) {
    if (elem) {
      G[tid] = grad;
      if (a.mode == 1) {
        B[tid] = pos;
        static_cast<T*>(a.eta)[tid] = mom;
      }
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
  if (elem) {
    if (acc) {
      B[tid] = pos;
      G[tid] = grad;
    }
    if (a.sample && rec) static_cast<T*>(a.sample)[t * pk + tid] = acc ? pos : b0;
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

template <typename T, int FP, int TH>
hipError_t launch_one(const TinyArgs& a, size_t lds, hipStream_t s) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tiny_kernel<T, FP, TH>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((tiny_kernel<T, FP, TH>), dim3(1), dim3(TH), lds, s, a);
  return hipGetLastError();
}

}  // namespace

// Where one workgroup beats the general path's kernels. Both times are near linear, here in us as
// measured in a graph at 400 sizes (f = padded free classes; p f <= 512 leaves a thread two gradient
// shares at most, and beyond it both the time and its spread double); the rule asks for 10% less
// per update and 5% less per gradient. Per update in FP32: p = 64 at n = 100, K = 3: 4.3 against
// 6.6; p = 128: 7.6 against 6.7, not taken. Per gradient: p = 20 at n = 500, K = 3, FP64: 9.7 against
// 10.3 in a graph and 11.3 launched singly; p = 256 at n = 100, K = 1: 21.7 against 9.6, not taken.
// A gradient launched singly is the faster one at every size taken, by 1 to 4 us of 10, since the
// general path's three launches pace it. In a graph it is at seven in eight: the model is off for 10
// or more classes in FP64 (n = 51, p = 2, K = 15: 8.9 against 8.1 in a graph, 9.0 against 10.2
// singly) and for one class of some 50 columns (n = 204, p = 50, K = 2, FP32: 9.2 against 7.9).
bool tiny_fits(int64_t n, int64_t p, int K, bool pin, bool f64, bool update) {
  if (n > 1024 || p > 256 || K > 16 || p * K > 1024 || n * p * K > (int64_t)1 << 16) return false;
  const int fp = class_pad(pin ? K - 1 : K);
  if (p * fp > 512 || (fp == 16 && n > 512)) return false;   // 16 classes: 512 threads (the times below say no more)
  const double N = (double)n, P = (double)p, F = fp, far = p > 128 ? 1.2 : 0.0;   // far: a wider row tile
  const double here =
      update ? (f64 ? 1.7 + P * (0.024 + 0.0116 * F) + N * (0.0010 + 0.00125 * F)
                    : 1.3 + P * (0.030 + 0.0078 * F) + N * (0.0016 + 0.00063 * F))
             : (f64 ? 5.4 + P * (0.034 + 0.0133 * F) + N * (0.0037 + 0.00122 * F)
                    : 5.0 + P * (0.035 + 0.0100 * F) + N * (0.0042 + 0.00061 * F));
  const double general = update ? (f64 ? 6.4 + 0.0046 * N : 6.1 + 0.0023 * N) + far
                                : (f64 ? 8.4 + 0.0044 * N : 8.3 + 0.0022 * N) + far;
  if (here * (update ? 1.10 : 1.05) > general) return false;
  return tiny_layout((int)n, (int)p, fp, tiny_threads(n, p * K), f64 ? 8 : 4).total <= kTinyLds;
}

template <typename T>
hipError_t launch_tiny(const TinyArgs& a, hipStream_t s) {
  const int fp = class_pad(a.pin ? a.K - 1 : a.K), th = tiny_threads(a.n, (int64_t)a.p * a.K);
  const size_t lds = tiny_layout((int)a.n, a.p, fp, th, sizeof(T)).total;
#define HMC_TINY(FP_)                                                                        \
  if (fp == FP_) return th == 512 ? launch_one<T, FP_, 512>(a, lds, s) : launch_one<T, FP_, 1024>(a, lds, s);
  HMC_TINY(1) HMC_TINY(2) HMC_TINY(4) HMC_TINY(8)
#undef HMC_TINY
  if (fp == 16 && th == 512) return launch_one<T, 16, 512>(a, lds, s);
  return hipErrorInvalidValue;
}

template hipError_t launch_tiny<float>(const TinyArgs&, hipStream_t);
template hipError_t launch_tiny<double>(const TinyArgs&, hipStream_t);

}  // namespace hmcx
