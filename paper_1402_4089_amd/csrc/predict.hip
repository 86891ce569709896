// Posterior-predictive classification (Section 3.2): for each row x_i of a data set, the
// mean over S coefficient samples B_s of the class probabilities softmax(x_i^T B_s),
// accumulated in float64, and the class of highest mean probability.
//
// The logits are a product of X with the p x (S K) matrix of all samples: 2 n p S (K - 1)
// operations against n p elements of X, so the matrix cores bound it (n = 10000, p = 785,
// K = 10, S = 100: 14 Gflop, 90 us at the FP32 matrix rate, against 5 us for the bytes). One
// workgroup per 16-row tile: the tile is staged in LDS once, and the waves share out the
// samples, so a wave streams each of its samples' coefficients (from the L2, which holds all
// of them) past the tile once. v_mfma 16x16x4 adds its four products one fused
// multiply-add after the other in the order of k, so with the columns of X taken four at a
// time in order a logit is the plain sum over j = 0, 1, .., p - 1 in the precision of X.
// Two layouts of the 16 output columns of a matrix instruction:
//   K <= 16  column = sample, one block per class: no column is spent on padding classes (nor
//            on the pinned class, whose logit is zero), and a lane holds all the classes of
//            its (row, sample), so the softmax needs no other lane;
//   K > 16   column = class, ceil(K / 16) blocks for each of two samples at a time: the first
//            layout would need 4 K accumulators per lane and more.
// Measured at the size above: 287 us, against 7990 us with the logits on the vector unit (each
// sample's coefficients staged in LDS by every tile, one multiply-add per two LDS reads).
// Few samples leave columns of the matrix and waves without work, and the registers leave a
// compute unit one to three workgroups; the vector-unit form (predict_rows) then stays, where
// rows_faster says so: n = 16607, p = 41, K = 14, S = 1 takes 7.1 us there and 65.4 here.
#include <math.h>

#include <algorithm>

#include "device_common.h"

namespace hmcx {
namespace {

using namespace dev;

// Steps of four columns whose coefficients are loaded as one group, a group ahead of the
// matrix instructions that use it: `w` 32-bit registers per step and lane. Enough that the
// instructions of a group cover a load's latency, few enough that two groups, the
// accumulators and the float64 sums fit the registers.
constexpr int group_steps(int w) { return w <= 2 ? 16 : w <= 4 ? 8 : w <= 10 ? 4 : w <= 16 ? 2 : 1; }

// Elements between two rows of the staged tile: whole groups, and an odd number of 16-byte
// pieces, so that the 16 rows of a read fall in different banks.
constexpr int64_t tile_pitch(int64_t p, size_t ts) { return (p + 63) / 64 * 64 + 16 / (int64_t)ts; }

template <typename T> __device__ __forceinline__ T buf1(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <> __device__ __forceinline__ float buf1<float>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
template <> __device__ __forceinline__ double buf1<double>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}

// N consecutive elements in as few loads as they take.
template <typename T, int N>
__device__ __forceinline__ void buf_run(__amdgpu_buffer_rsrc_t r, uint32_t off, T (&v)[N]) {
  constexpr int E = 16 / sizeof(T);
  typedef T vec_t __attribute__((ext_vector_type(E)));
  int f = 0;
#pragma unroll
  for (; f + E <= N; f += E) {
    const vec_t q = __builtin_bit_cast(
        vec_t, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off + f * (int)sizeof(T)), 0, 0));
#pragma unroll
    for (int e = 0; e < E; ++e) v[f + e] = q[e];
  }
  if constexpr (sizeof(T) == 4) {
    if constexpr (N % 4 >= 2) {
      typedef float f2 __attribute__((ext_vector_type(2)));
      const f2 q = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)(off + f * 4), 0, 0));
      v[f] = q[0]; v[f + 1] = q[1];
      f += 2;
    }
  }
  if constexpr (N % 2 == 1) v[f] = buf1<T>(r, off + f * (int)sizeof(T));
}

// Rows [i0, i0 + 16) of X into LDS, zero past row n and column p. Inside a group of 16 columns
// column 4 s + g is stored at 4 g + s: the elements that lane group g feeds to four steps are
// then one 16-byte read (32 for float64). rowbad[r] is set if row r holds an infinity or a NaN.
template <typename T>
__device__ __forceinline__ void stage_tile(const PredictArgs& a, int64_t i0, T* xs, int64_t pitch, int* rowbad) {
  const T* X = static_cast<const T*>(a.X);
  if (threadIdx.x < 16) rowbad[threadIdx.x] = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int cols = (a.p + 63) / 64 * 64;
  for (int r = threadIdx.x >> 6; r < 16; r += nw) {
    const bool row = i0 + r < a.n;
    bool bad = false;
    for (int j = lane; j < cols; j += 64) {
      const T x = (row && j < a.p) ? X[(i0 + r) * a.ldx + j] : T(0);
      bad |= !(x * T(0) == T(0));
      xs[r * pitch + (j & ~15) + 4 * (j & 3) + ((j >> 2) & 3)] = x;
    }
    if (bad) rowbad[r] = 1;
  }
  __syncthreads();
}

// The A operands of G steps from step s0 (a multiple of G): lane 16 g + c holds row c's column
// 4 s + g of step s.
template <typename T, int G>
__device__ __forceinline__ void tile_operands(const T* xs, int64_t pitch, int s0, int g, int c, T (&av)[G]) {
  const T* x = xs + c * pitch + (s0 >> 2) * 16 + 4 * g + (s0 & 3);
#pragma unroll
  for (int s = 0; s < G; ++s) av[s] = x[(s >> 2) * 16 + (s & 3)];
}

// Mean probabilities and classes of the tile from the waves' sums red[wave][row][16 NB].
template <int NB>
__device__ __forceinline__ void finish_tile(const PredictArgs& a, int64_t i0, const double* red) {
  if (threadIdx.x >= 256) return;
  const int nw = blockDim.x >> 6, r = threadIdx.x >> 4, c = threadIdx.x & 15, K = a.K;
  const int64_t i = i0 + r;
  const double inv = 1.0 / (double)a.n_samples;
  double best = -1.0;
  int bk = 0;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int k = 16 * q + c;
    double m = 0.0;
    for (int w = 0; w < nw; ++w) m += red[(w * 16 + r) * (16 * NB) + k];
    m *= inv;
    if (k < K && i < a.n && a.mean_prob) a.mean_prob[i * K + k] = m;
    if (k < K && m > best) { best = m; bk = k; }
  }
  // argmax across the 16 lanes of the row: compare (value, -index) pairs
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    const double ob = __shfl_xor(best, m, 64);
    const int ok = __shfl_xor(bk, m, 64);
    if (ob > best || (ob == best && ok < bk)) { best = ob; bk = ok; }
  }
  if (c == 0 && i < a.n && a.classes) a.classes[i] = bk;
}

// Sum of 16 values in the order of a 16-lane DPP reduction (pairs, quads, halves).
template <typename T> __device__ __forceinline__ T tree16(const T (&e)[16]) {
  return (((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]))) +
         (((e[8] + e[9]) + (e[10] + e[11])) + ((e[12] + e[13]) + (e[14] + e[15])));
}

// Most waves of a workgroup. The two coefficient groups, the accumulators and the float64 sums
// of up to 9 classes (4 in float64) take 256 registers per lane (9 in float32 and 20 bytes of
// scratch), so two waves per SIMD and workgroups of 8 waves; more classes take the 512 of one wave
// per SIMD (14, 15 and 16 in float64 and 88, 216 and 220 bytes of scratch).
template <typename T, int F> constexpr int sample_waves() { return F <= (sizeof(T) == 4 ? 9 : 4) ? 8 : 4; }

// K <= 16: F classes with coefficients (K, or K - 1 with the pinned class last); lane 16 g + c
// holds sample c of a group of 16, block f is class f.
template <typename T, int F>
__global__ __launch_bounds__((64 * sample_waves<T, F>())) void predict_samples(PredictArgs a) {
  using M = Mma<T>;
  using acc_t = typename M::acc;
  constexpr int G = group_steps(F * (int)sizeof(T) / 4);
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int rowbad[16];
  T* xs = reinterpret_cast<T*>(smem);
  double* red = reinterpret_cast<double*>(smem);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int p = a.p, K = a.K;
  const bool pin = a.pin;
  const int64_t pitch = tile_pitch(p, sizeof(T)), pk = (int64_t)p * K;
  const int nsteps = (p + 3) / 4, ngrp = (nsteps + G - 1) / G, nsg = (a.n_samples + 15) / 16;
  const uint32_t voff = (uint32_t)((c * pk + g * K) * sizeof(T));
  for (int64_t tile = blockIdx.x; tile * 16 < a.n; tile += gridDim.x) {
    const int64_t i0 = tile * 16;
    stage_tile<T>(a, i0, xs, pitch, rowbad);
    double sum[4][F + 1];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int f = 0; f <= F; ++f) sum[r][f] = 0.0;
    // the waves' shares differ by one group of samples at most; the tile index turns them, so
    // that the longer shares of a compute unit's workgroups fall to different SIMDs
    for (int sg = (w + (int)(tile % nw)) % nw; sg < nsg; sg += nw) {
      const int left = a.n_samples - 16 * sg;
      const __amdgpu_buffer_rsrc_t br = make_rsrc(static_cast<const T*>(a.samples) + 16 * sg * pk,
                                                  (uint64_t)(left < 16 ? left : 16) * pk * sizeof(T));
      // coefficients of steps s0 .. s0 + G - 1; a row at or past p, and a sample past the last,
      // loads from past the resource's end: zeros
      auto load = [&](int s0, T (&b)[G][F]) {
#pragma unroll
        for (int s = 0; s < G; ++s)
          buf_run<T, F>(br, 4 * (s0 + s) + g < p ? voff + (uint32_t)(4 * (s0 + s) * K * (int)sizeof(T))
                                                 : 0x40000000u, b[s]);
      };
      acc_t acc[F];
#pragma unroll
      for (int f = 0; f < F; ++f) acc[f] = acc_t{0, 0, 0, 0};
      auto mma = [&](int s0, const T (&b)[G][F]) {
        T av[G];
        tile_operands<T, G>(xs, pitch, s0, g, c, av);
#pragma unroll
        for (int s = 0; s < G; ++s)
#pragma unroll
          for (int f = 0; f < F; ++f) acc[f] = M::run(av[s], b[s][f], acc[f]);
      };
      T b0[G][F], b1[G][F];
      load(0, b0);
      for (int q = 0; q < ngrp; q += 2) {
        load((q + 1) * G, b1);
        mma(q * G, b0);
        if (q + 1 >= ngrp) break;
        load((q + 2) * G, b0);
        mma((q + 1) * G, b1);
      }
      // softmax over the classes of (row r, this lane's sample); the pinned class's logit is
      // the sum of x * 0: zero, or a NaN in a row that holds an infinity or a NaN
      const bool real = 16 * sg + c < a.n_samples;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const T zpin = rowbad[M::row(r, g)] ? (T)NAN : T(0);
        T mx = acc[0][r];
#pragma unroll
        for (int f = 1; f < F; ++f) mx = fmax(mx, acc[f][r]);
        if (pin) mx = fmax(mx, zpin);
        T e[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) e[k] = T(0);
#pragma unroll
        for (int f = 0; f < F; ++f) e[f] = exp(acc[f][r] - mx);
        if constexpr (F < 16) e[F] = pin ? exp(zpin - mx) : T(0);
        const double inv = 1.0 / (double)tree16(e);
#pragma unroll
        for (int f = 0; f < F + (F < 16); ++f) sum[r][f] += real ? (double)e[f] * inv : 0.0;
      }
    }
    __syncthreads();                                        // the tile is read: its LDS takes the sums
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int f = 0; f < F + (F < 16); ++f) {
        const double v = sum16(sum[r][f]);
        if (c == f) red[(w * 16 + M::row(r, g)) * 16 + f] = v;
      }
    __syncthreads();
    finish_tile<1>(a, i0, red);
    __syncthreads();
  }
}

// K > 16: lane 16 g + c holds class 16 q + c of block q, two samples at a time.
template <typename T, int NB>
__global__ __launch_bounds__(256) void predict_classes(PredictArgs a) {
  using M = Mma<T>;
  using acc_t = typename M::acc;
  constexpr int G = sizeof(T) == 4 ? 4 : 2;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int rowbad[16];
  T* xs = reinterpret_cast<T*>(smem);
  double* red = reinterpret_cast<double*>(smem);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int p = a.p, K = a.K, kmax = a.pin ? K - 1 : K;
  const int64_t pitch = tile_pitch(p, sizeof(T)), pk = (int64_t)p * K;
  const int nsteps = (p + 3) / 4, ngrp = (nsteps + G - 1) / G, nsp = (a.n_samples + 1) / 2;
  for (int64_t tile = blockIdx.x; tile * 16 < a.n; tile += gridDim.x) {
    const int64_t i0 = tile * 16;
    stage_tile<T>(a, i0, xs, pitch, rowbad);
    double sum[4][NB];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < NB; ++q) sum[r][q] = 0.0;
    for (int sp = (w + (int)(tile % nw)) % nw; sp < nsp; sp += nw) {
      const int left = a.n_samples - 2 * sp;
      const __amdgpu_buffer_rsrc_t br = make_rsrc(static_cast<const T*>(a.samples) + 2 * sp * pk,
                                                  (uint64_t)(left < 2 ? left : 2) * pk * sizeof(T));
      // a class past the free ones, a row at or past p and a sample past the last load zeros
      auto load = [&](int s0, T (&b)[G][2][NB]) {
#pragma unroll
        for (int s = 0; s < G; ++s)
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < NB; ++q) {
              const int j = 4 * (s0 + s) + g, k = 16 * q + c;
              b[s][u][q] = buf1<T>(br, (j < p && k < kmax) ? (uint32_t)((u * pk + (int64_t)j * K + k) * sizeof(T))
                                                           : 0x40000000u);
            }
      };
      acc_t acc[2][NB];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int q = 0; q < NB; ++q) acc[u][q] = acc_t{0, 0, 0, 0};
      auto mma = [&](int s0, const T (&b)[G][2][NB]) {
        T av[G];
        tile_operands<T, G>(xs, pitch, s0, g, c, av);
#pragma unroll
        for (int s = 0; s < G; ++s)
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < NB; ++q) acc[u][q] = M::run(av[s], b[s][u][q], acc[u][q]);
      };
      T b0[G][2][NB], b1[G][2][NB];
      load(0, b0);
      for (int q = 0; q < ngrp; q += 2) {
        load((q + 1) * G, b1);
        mma(q * G, b0);
        if (q + 1 >= ngrp) break;
        load((q + 2) * G, b0);
        mma((q + 1) * G, b1);
      }
      // softmax over the K classes of row r: max and sum over the 16 lanes of the row
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // the pinned class's logit: zero, or a NaN in a row that holds an infinity or a NaN
          const T zpin = rowbad[M::row(r, g)] ? (T)NAN : T(0);
          T z[NB], e[NB], mx = -INFINITY, se = T(0);
#pragma unroll
          for (int q = 0; q < NB; ++q) {
            const int k = 16 * q + c;
            z[q] = k < kmax ? acc[u][q][r] : zpin;
            if (k < K) mx = fmax(mx, z[q]);
          }
          mx = max16(mx);
#pragma unroll
          for (int q = 0; q < NB; ++q) {
            e[q] = 16 * q + c < K ? exp(z[q] - mx) : T(0);
            se += e[q];
          }
          const double inv = 1.0 / (double)sum16(se);
#pragma unroll
          for (int q = 0; q < NB; ++q) sum[r][q] += 2 * sp + u < a.n_samples ? (double)e[q] * inv : 0.0;
        }
    }
    __syncthreads();                                        // the tile is read: its LDS takes the sums
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < NB; ++q) red[(w * 16 + M::row(r, g)) * (16 * NB) + 16 * q + c] = sum[r][q];
    __syncthreads();
    finish_tile<NB>(a, i0, red);
    __syncthreads();
  }
}

// Few samples, or rows of a few columns and many tiles: thread (r, c) = (tid / 16, tid % 16) of a
// 16-row tile forms the logits of row r for classes c, c + 16, .. of one sample after the other, whose
// coefficients are staged in LDS in turn (the 16 lanes of a row are one DPP row). Two LDS reads
// per multiply-add bound it; eight workgroups fit a compute unit while the LDS holds them.
template <typename T, int NB>
__global__ __launch_bounds__(256) void predict_rows(PredictArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  T* xs = reinterpret_cast<T*>(smem);                       // [16][p]
  T* bs = xs + 16 * (int64_t)a.p;                           // [p][K] of the current sample
  const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
  const int p = a.p, K = a.K;
  const int kmax = a.pin ? K - 1 : K;
  const int64_t n = a.n, ldx = a.ldx;
  const T* X = static_cast<const T*>(a.X);
  const T* S = static_cast<const T*>(a.samples);
  const int64_t pk = (int64_t)p * K;
  for (int64_t tile = blockIdx.x; tile * 16 < n; tile += gridDim.x) {
    const int64_t i0 = tile * 16;
    __syncthreads();                                        // previous tile's readers done
    for (int64_t e = tid; e < 16 * (int64_t)p; e += 256) {
      const int64_t rr = e / p, j = e - rr * p;
      xs[e] = (i0 + rr < n) ? X[(i0 + rr) * ldx + j] : T(0);
    }
    double acc[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) acc[q] = 0.0;
    for (int s = 0; s < a.n_samples; ++s) {
      __syncthreads();                                      // previous sample's readers done
      const T* Bs = S + (int64_t)s * pk;
      for (int64_t e = tid; e < pk; e += 256) bs[e] = Bs[e];
      __syncthreads();
      T z[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) z[q] = T(0);
      const T* xr = xs + (int64_t)r * p;
      for (int j = 0; j < p; ++j) {
        const T xv = xr[j];
        const T* br = bs + (int64_t)j * K;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          const int k = 16 * q + c;
          z[q] += xv * (k < kmax ? br[k] : T(0));
        }
      }
      // softmax over the K classes of row r (the pinned class, if any, keeps logit 0)
      T mx = -INFINITY;
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (16 * q + c < K) mx = fmax(mx, z[q]);
      mx = max16(mx);
      T ex[NB], se = T(0);
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        ex[q] = (16 * q + c < K) ? exp(z[q] - mx) : T(0);
        se += ex[q];
      }
      se = sum16(se);
#pragma unroll
      for (int q = 0; q < NB; ++q) acc[q] += (double)ex[q] / (double)se;
    }
    // mean probabilities and the class of the largest (lowest index among exact ties)
    const int64_t i = i0 + r;
    const double inv = 1.0 / (double)a.n_samples;
    double best = -1.0;
    int bk = 0;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int k = 16 * q + c;
      const double m = acc[q] * inv;
      if (k < K && i < n && a.mean_prob) a.mean_prob[i * K + k] = m;
      if (k < K && m > best) { best = m; bk = k; }
    }
    // argmax across the 16 lanes of the row: compare (value, -index) pairs
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) {
      const double ob = __shfl_xor(best, m, 64);
      const int ok = __shfl_xor(bk, m, 64);
      if (ob > best || (ob == best && ok < bk)) { best = ob; bk = ok; }
    }
    if (c == 0 && i < n && a.classes) a.classes[i] = bk;
  }
}

template <typename T, int NB>
hipError_t launch_rows(const PredictArgs& a, hipStream_t s) {
  const int64_t tiles = (a.n + 15) / 16;
  const size_t lds = predict_lds_bytes(a.p, a.K, sizeof(T) == 8);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&predict_rows<T, NB>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((predict_rows<T, NB>), dim3((unsigned)(tiles < 16384 ? tiles : 16384)), dim3(256), lds, s, a);
  return hipGetLastError();
}

size_t matrix_lds(int64_t p, int waves, int nb, size_t ts) {
  const size_t tile = 16 * (size_t)tile_pitch(p, ts) * ts, sums = (size_t)waves * 16 * 16 * nb * 8;
  return tile > sums ? tile : sums;
}

template <typename KERN>
hipError_t launch_kernel(KERN kernel, const PredictArgs& a, int waves, int nb, size_t ts, hipStream_t s) {
  const size_t lds = matrix_lds(a.p, waves, nb, ts);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int64_t tiles = (a.n + 15) / 16;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(tiles < (1 << 20) ? tiles : (1 << 20))), dim3(64 * waves), lds, s, a);
  return hipGetLastError();
}

// Is the vector-unit form the faster one? Both times follow from a tile's and the workgroups that a
// compute unit holds at once, here in us as fitted to 6400 sizes (n <= 400000, p <= 2200, up to 200
// samples; 90% within 20%), so that the choice is slower than the other form by more than 3% at 2%
// of them. With u tiles per compute unit, w workgroups of the form at once, f blocks of a matrix step
// (free classes up to 16 classes, then 16 classes each) and g turns of a wave's sample groups:
//   rows    3.3 + (r4 p + S (r0 + r1 p ceil(K / 16) + r2 p K)) (max(1, u / w) + r3 u)
//   matrix  m0 + (m1 f + g (m2 + m3 f + ceil(p / 4) (m4 + m5 f))) ceil(u / w) (1 + m6 (min(u, w) - 1))
// The rows also get what they lose by less than 5% (10% beyond 16 classes), about what the fit is
// off where the two cross.
struct FormTimes { double r[5], m[7]; };
constexpr FormTimes kFormTimes[2][2] = {
  {{{0.343, 0.0376, 0.00041, 0.104, 0.0189}, {1.82, 0.384, 3.44, 0.0, 0.0542, 0.0243, 0.149}},
   {{0.386, 0.0203, 0.00056, 0.135, 0.0119}, {3.46, 0.641, 0.958, 0.470, 0.0349, 0.0724, 0.415}}},
  {{{0.456, 0.0407, 0.00033, 0.157, 0.0226}, {2.07, 0.533, 3.06, 0.0508, 0.0221, 0.0506, 0.267}},
   {{0.568, 0.0177, 0.00084, 0.223, 0.0112}, {2.70, 0.881, 1.14, 0.845, 0.0731, 0.0963, 0.435}}}};

bool rows_faster(const PredictArgs& a, bool f64) {
  const size_t ts = f64 ? 8 : 4;
  const bool wide = a.K > 16;
  const FormTimes& t = kFormTimes[f64][wide];
  const int nb = (a.K + 15) / 16, F = a.pin ? a.K - 1 : a.K;
  const int most = F <= (f64 ? 4 : 9) ? 8 : 4, waves = !wide && a.n_samples > 64 ? most : 4;
  // waves per SIMD that the matrix form's registers allow
  const int occ = wide ? (nb <= (f64 ? 2 : 3) ? 2 : 1) : !f64 && F <= 3 ? 3 : F <= (f64 ? 4 : 9) ? 2 : 1;
  const double p = a.p, S = a.n_samples, u = (double)((a.n + 15) / 16) / 256.0, f = wide ? nb : F;
  const double lds = 160.0 * 1024.0;
  const double wr = std::clamp(floor(lds / (double)(predict_lds_bytes(a.p, a.K, f64) + 1)), 1.0, 8.0);
  const double wm = std::max(1.0, std::min((double)(4 * occ / waves), floor(lds / (double)(matrix_lds(a.p, waves, wide ? nb : 1, ts) + 64))));
  const double g = ceil(ceil(S / (wide ? 2.0 : 16.0)) / waves), u1 = std::max(u, 1.0);
  const double rows = 3.3 + (t.r[4] * p + S * (t.r[0] + t.r[1] * p * nb + t.r[2] * p * a.K)) * (std::max(1.0, u / wr) + t.r[3] * u);
  const double matrix = t.m[0] + (t.m[1] * f + g * (t.m[2] + t.m[3] * f + ceil(p / 4.0) * (t.m[4] + t.m[5] * f))) *
                                     ceil(u1 / wm) * (1.0 + t.m[6] * (std::min(u1, wm) - 1.0));
  return rows < (wide ? 1.10 : 1.05) * matrix;
}

// Eight waves where two fit a SIMD and there are more than four groups of samples to share out.
template <typename T, int F>
hipError_t launch_samples(const PredictArgs& a, hipStream_t s) {
  const int waves = a.n_samples > 64 ? sample_waves<T, F>() : 4;
  return launch_kernel(&predict_samples<T, F>, a, waves, 1, sizeof(T), s);
}

}  // namespace

// A 16-row tile and one sample: what predict_rows holds, and the bound of the call. It leaves p <= 2275
// in FP32 and 1137 in FP64, so the matrix forms' tile of whole 64-column groups takes 148 KB at most.
size_t predict_lds_bytes(int64_t p, int K, bool f64) {
  return (size_t)(16 * p + p * K) * (f64 ? 8 : 4);
}

template <typename T>
hipError_t launch_predict(const PredictArgs& a, hipStream_t s) {
  if (rows_faster(a, sizeof(T) == 8)) {
    switch ((a.K + 15) / 16) {
      case 1: return launch_rows<T, 1>(a, s);
      case 2: return launch_rows<T, 2>(a, s);
      case 3: return launch_rows<T, 3>(a, s);
      case 4: return launch_rows<T, 4>(a, s);
    }
  }
  if (a.K <= 16) {
    switch (a.pin ? a.K - 1 : a.K) {
#define HMC_PRED(F_) case F_: return launch_samples<T, F_>(a, s);
      HMC_PRED(1) HMC_PRED(2) HMC_PRED(3) HMC_PRED(4) HMC_PRED(5) HMC_PRED(6) HMC_PRED(7) HMC_PRED(8)
      HMC_PRED(9) HMC_PRED(10) HMC_PRED(11) HMC_PRED(12) HMC_PRED(13) HMC_PRED(14) HMC_PRED(15) HMC_PRED(16)
#undef HMC_PRED
    }
  } else {
    switch ((a.K + 15) / 16) {
#define HMC_PRED(NB_) case NB_: return launch_kernel(&predict_classes<T, NB_>, a, 4, NB_, sizeof(T), s);
      HMC_PRED(2) HMC_PRED(3) HMC_PRED(4)
#undef HMC_PRED
    }
  }
  return hipErrorInvalidValue;
}

template hipError_t launch_predict<float>(const PredictArgs&, hipStream_t);
template hipError_t launch_predict<double>(const PredictArgs&, hipStream_t);

}  // namespace hmcx
