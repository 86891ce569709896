// Log-posterior + gradient for p too wide for one compute unit's row tile (p >> n).
//
// Same quantities as the fused pass (Section 2.1: logits X B, row softmax and
// log-likelihood, gradient X^T (Y - psi(XB)) plus the prior term), split into three
// kernels because a row's logits need all p columns before its residuals exist:
//   wide_logits   16-row x 1024-column blocks of X on MFMA -> per-chunk partial logits
//   wide_softmax  sums the chunk partials of a row, softmax, residuals R, log-likelihood
//   wide_grad     each wave owns 256 bytes of columns, streams the rows of X and R (all of
//                 them, or one row slice) through MFMA (G block = X^T R); with all rows it
//                 then applies prior, mask and the leapfrog kicks and drift to its own
//                 columns (no cross-workgroup reduction), with row slices it writes partials
//                 for the shared epilogue.
// X is read twice per gradient, which bounds the path: the matrix cores are busy a third of the
// time. All loads go through buffer resources whose bounds make rows past n read as zero.
#include <type_traits>

#include "device_common.h"

namespace hmcx {

using namespace dev;

namespace {

constexpr int kWideWaves = 4;

// Columns of a logits workgroup.
template <typename T> constexpr int wide_chunk() { return kWideWaves * (sizeof(T) == 4 ? 16 : 8) * 16; }

// 16 bytes of X or R: 4 floats or 2 doubles.
template <typename T> using vec16 = T __attribute__((ext_vector_type(16 / sizeof(T))));
template <typename T> __device__ __forceinline__ vec16<T> ld16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(vec16<T>, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}

// Partial logits over one column chunk for the row tiles tile0, tile0 + tstep, ...
// Wave w covers columns [chunk*CW + w*MBW*16, ... + MBW*16) in MBW blocks of 16. The chunk is
// the fast grid dimension, so the workgroups running together read the same rows (measured:
// with the chunk as the slow dimension the pass at n = 2000, p = 50000 took about 4% longer).
template <typename T, int NB>
__global__ __launch_bounds__(kWideWaves * 64) void wide_logits(WideArgs a) {
  using M = Mma<T>;
  using acc_t = typename M::acc;
  constexpr int MBW = sizeof(T) == 4 ? 16 : 8;
  constexpr int CW = wide_chunk<T>();
  __shared__ __align__(16) T zb[kWideWaves * NB * 256];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int p = a.p, K = a.K;
  const int64_t n = a.n, ldx = a.ldx;
  const int chunk = blockIdx.x;
  const int jw = chunk * CW + w * MBW * 16;              // first column of this wave
  const T* B = static_cast<const T*>(a.B);

  // the pinned column is read as zero (beta_K = 0 in the model)
  const int kmax = a.pin ? K - 1 : K;
  T bt[MBW][NB][4];
#pragma unroll
  for (int m = 0; m < MBW; ++m)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int j = jw + m * 16 + 4 * g + t, k = nb * 16 + c;
        bt[m][nb][t] = (j < p && k < kmax) ? B[(int64_t)j * K + k] : T(0);
      }
  const bool maskcols = ldx != p && jw + MBW * 16 > p;   // row padding inside this wave's span
  const uint64_t x_bytes = (uint64_t)((n - 1) * ldx + p) * sizeof(T);

  for (int64_t tile = blockIdx.y; tile * kTileRows < n; tile += gridDim.y) {
    const int64_t i0 = tile * kTileRows;
    const uint64_t base = (uint64_t)i0 * ldx * sizeof(T);
    const __amdgpu_buffer_rsrc_t xr =
        make_rsrc(static_cast<const char*>(a.X) + base, x_bytes - base);
    // A lane whose four columns all lie past p (the tail of the last chunk) loads from an
    // offset past the resource's end: zeros and no traffic where the rest of X is under 4 GB,
    // an in-bounds read of X's own elements otherwise (finite, and multiplied by coefficients
    // that are zero past p; with padded rows the wave's mask below zeroes them). Reading the
    // next rows there instead cost the last chunk as much traffic as a full one. The mask is
    // a wave-uniform branch: a per-lane one waits for each load before the next issues (2-7%
    // slower passes, measured).
    T av[MBW][4];
#pragma unroll
    for (int m = 0; m < MBW; ++m) {
      const int col0 = jw + m * 16 + 4 * g;
      const bool live = col0 < p;
      const uint32_t off = live ? (uint32_t)(((int64_t)c * ldx + col0) * sizeof(T)) : 0xFFFFFFE0u;
      if constexpr (sizeof(T) == 4) {
        const vec16<T> q = ld16<T>(xr, off);
        av[m][0] = q[0]; av[m][1] = q[1]; av[m][2] = q[2]; av[m][3] = q[3];
      } else {
        const vec16<T> q0 = ld16<T>(xr, off), q1 = ld16<T>(xr, off + 16);
        av[m][0] = q0[0]; av[m][1] = q0[1]; av[m][2] = q1[0]; av[m][3] = q1[1];
      }
      if (maskcols) {
#pragma unroll
        for (int t = 0; t < 4; ++t) av[m][t] = (col0 + t < p) ? av[m][t] : T(0);
      }
    }
    acc_t z0[NB], z1[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) z0[nb] = z1[nb] = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int m = 0; m < MBW; ++m)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          if (m & 1) z1[nb] = M::run(av[m][t], bt[m][nb][t], z1[nb]);
          else       z0[nb] = M::run(av[m][t], bt[m][nb][t], z0[nb]);
        }
    __syncthreads();                                      // previous tile's exchange read
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) zb[((nb * 4 + r) * kWideWaves + w) * 64 + lane] = z0[nb][r] + z1[nb][r];
    __syncthreads();
    if (w == 0) {
      T* zp = static_cast<T*>(a.zpart) + (int64_t)chunk * n * (16 * NB);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const T* src = zb + (nb * 4 + r) * kWideWaves * 64 + lane;
          const T v = ((src[0] + src[64]) + src[128]) + src[192];
          const int64_t i = i0 + M::row(r, g);
          if (i < n) zp[i * (16 * NB) + nb * 16 + c] = v;
        }
    }
  }
}

// Row softmax over the summed chunk partials: 4 rows per workgroup, 16 lanes per row. Wave g
// sums chunks g, g + 4, g + 8, ... of the four rows, the four sums are added in wave order
// through LDS, and wave 0 finishes the rows (a quarter of the dependent loads per thread of a
// one-wave-per-row-group form, whose chain over all chunks paced the kernel).
template <typename T, int NB>
__global__ __launch_bounds__(256) void wide_softmax(WideArgs a) {
  constexpr int KP = 16 * NB;
  __shared__ T zs[4][NB][64];
  const int tid = threadIdx.x, lane = tid & 63, grp = tid >> 6, c = lane & 15;
  const int K = a.K;
  const int64_t n = a.n;
  const int64_t i = (int64_t)blockIdx.x * 4 + (lane >> 4);
  const bool valid = i < n;
  const int64_t ic = valid ? i : n - 1;
  const T* zp = static_cast<const T*>(a.zpart) + ic * KP + c;
  T zz[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) zz[nb] = T(0);
#pragma unroll 4
  for (int ch = grp; ch < a.nchunk; ch += 4)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) zz[nb] += zp[(int64_t)ch * n * KP + nb * 16];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) zs[grp][nb][lane] = zz[nb];
  __syncthreads();
  if (grp != 0) return;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
    zz[nb] = ((zs[0][nb][lane] + zs[1][nb][lane]) + zs[2][nb][lane]) + zs[3][nb][lane];
  const int yi = a.y[ic];
  double l = 0.0;
  // residuals in the lane order of the gradient's B operand: [16-row tile][block][lane][step],
  // row M::row(s, g) of the tile at step s of lane 16 g + c; rows past n are zero
  const int rt = (int)(i & 15), rs = sizeof(T) == 4 ? rt & 3 : rt >> 2, rg = sizeof(T) == 4 ? rt >> 2 : rt & 3;
  T* R = static_cast<T*>(a.R) + ((i >> 4) * NB * 64 + 16 * rg + c) * 4 + rs;
  if (a.link == 1) {
    // Poisson link, one coefficient column (lane c = 0): residual y - exp(z), term y z - exp(z)
    const T mu = dev_exp(zz[0]);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int k = nb * 16 + c;
      R[nb * 256] = valid && k == 0 ? T(yi) - mu : T(0);
    }
    l = (valid && c == 0) ? (double)yi * (double)zz[0] - (double)mu : 0.0;
  } else if (a.link == 2) {
    // probit link, one coefficient column (lane c = 0): residual s phi(z) / Phi(s z) with
    // s = +1 for a success and -1 otherwise, term log Phi(s z)
    const T sg = yi == 1 ? T(1) : T(-1);
    T ratio;
    double lp;
    probit_row(sg * zz[0], ratio, lp);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int k = nb * 16 + c;
      R[nb * 256] = valid && k == 0 ? sg * ratio : T(0);
    }
    l = (valid && c == 0) ? lp : 0.0;
  } else {
    T mx = -INFINITY;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      if (nb * 16 + c < K) mx = fmax(mx, zz[nb]);
    mx = max16(mx);
    T ex[NB], se = T(0);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      ex[nb] = (nb * 16 + c < K) ? dev_exp(zz[nb] - mx) : T(0);
      se += ex[nb];
    }
    se = sum16(se);
    const T inv = dev_rcp(se);
    const T lse_shift = dev_log(se);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int k = nb * 16 + c;
      const bool hit = valid && k == yi;
      R[nb * 256] = valid && k < K ? ((hit ? T(1) : T(0)) - ex[nb] * inv) : T(0);
      l += hit ? (double)((zz[nb] - mx) - lse_shift) : 0.0;
    }
  }
  l = wave_sum(l);
  if (lane == 0) a.lpart[blockIdx.x] = l;
}

// W consecutive elements at a byte offset: one, or those of 16 bytes.
template <typename T, int W> struct Run { typedef vec16<T> type; };
template <typename T> struct Run<T, 1> { typedef T type; };
template <typename T, int W>
__device__ __forceinline__ typename Run<T, W>::type ld_run(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (W > 1) return ld16<T>(r, off);
  else if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
  else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}
template <typename V> __device__ __forceinline__ auto run_elem(const V& v, int e) {
  if constexpr (std::is_arithmetic_v<V>) return v;
  else return v[e];
}

// Column-owner gradient. A wave owns 256 bytes of a row, 16 E consecutive columns. A lane's 16-byte load
// takes E consecutive columns of one row; as which column of G a row of the MFMA's output means
// is free, element e of the load is the A operand of a block that holds columns E c + e, c = 0
// .. 15: one instruction reads 4 rows x 256 bytes and feeds E blocks (loads of one element per
// lane had taken E times the instructions, of 64 bytes per row). With one row slice (gridDim.y
// == 1) the workgroup applies the leapfrog epilogue to its own columns; with several, slice
// blockIdx.y covers tiles_per_split 16-row tiles (a multiple of the U-tile load group) and writes
// its partial X^T R to gpart for the shared epilogue kernel. Measured against one element per
// lane: n = 2000, p = 50000, K = 4, FP32 75.5 -> 71.4 us (5.6 TB/s); a whole gradient of
// n = 5000, p = 1000, K = 10, FP64 46 -> 33 us, n = 2000, p = 10000, K = 4, FP64 84 -> 64 us.
// W: elements of a load, E, or 1 (16 columns per wave) where the wider spans leave compute units
// idle and each wave E times the matrix instructions.
template <typename T, int NB, int W>
__global__ __launch_bounds__(kWideWaves * 64, (sizeof(T) * NB <= 8 ? 3 : sizeof(T) * NB <= 16 ? 2 : 1)) void wide_grad(WideArgs a) {
  __shared__ double sh4[2][4];
  using M = Mma<T>;
  using acc_t = typename M::acc;
  constexpr int E = 16 / sizeof(T), U = 2;               // U row tiles per load group
  constexpr int RB = 4 / E;                              // 16-byte loads of a tile's residual operand
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int p = a.p, K = a.K;
  const int64_t n = a.n, ldx = a.ldx;
  const int j0 = ((int)blockIdx.x * kWideWaves + w) * 16 * W;   // first column of this wave

  const uint64_t x_bytes = (uint64_t)((n - 1) * ldx + p) * sizeof(T);
  acc_t gacc[W][NB];
#pragma unroll
  for (int e = 0; e < W; ++e)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) gacc[e][nb] = acc_t{0, 0, 0, 0};
  const int64_t ntiles = (n + kTileRows - 1) / kTileRows;
  const int64_t tbeg = (int64_t)blockIdx.y * a.tiles_per_split;
  const int64_t tend = gridDim.y == 1 ? ntiles : (tbeg + a.tiles_per_split < ntiles ? tbeg + a.tiles_per_split : ntiles);
  const int64_t ngroups = tend > tbeg ? (tend - tbeg + U - 1) / U : 0;

  // Groups of U row tiles are visited last to first: the logits pass has just read the
  // last rows of X, so the first groups here may still be held by the memory-side cache.
  // Group k - 1 is loaded while group k is multiplied; a group index below 0 gets
  // resources without records, so its loads return zeros without touching memory and
  // the issue stays free of branches. A lane whose columns lie past p loads from an
  // offset past every resource's end: zeros, no traffic (columns past p only feed columns of
  // G that are not written).
  struct Regs { typename Run<T, W>::type xa[U][4]; vec16<T> ra[U][NB][RB]; };
  const bool live = j0 + c * W < p;
  uint32_t xoff[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) xoff[s] = (uint32_t)(((int64_t)M::row(s, g) * ldx + j0 + c * W) * sizeof(T));
  const uint32_t xstep = (uint32_t)(kTileRows * ldx * sizeof(T));
  auto load = [&](int64_t k, Regs& rg) {
    const bool real = k >= 0;
    const int64_t t0 = tbeg + (real ? k : 0) * U;
    const uint64_t base = (uint64_t)(t0 * kTileRows) * ldx * sizeof(T);
    const uint64_t rbase = (uint64_t)t0 * NB * 256 * sizeof(T), rall = (uint64_t)ntiles * NB * 256 * sizeof(T);
    const __amdgpu_buffer_rsrc_t xr =
        make_rsrc(static_cast<const char*>(a.X) + base, real ? x_bytes - base : 0);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(static_cast<const char*>(a.R) + rbase, real ? rall - rbase : 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // the second tile of a slice's odd count belongs to the next slice: not read
      const bool in = t0 + u < tend;
#pragma unroll
      for (int s = 0; s < 4; ++s) rg.xa[u][s] = ld_run<T, W>(xr, in && live ? xoff[s] + u * xstep : 0xFFFFFFF0u);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int q = 0; q < RB; ++q)
          rg.ra[u][nb][q] = ld16<T>(rr, in ? (uint32_t)((((u * NB + nb) * 64 + lane) * RB + q) * 16) : 0xFFFFFFF0u);
    }
  };
  auto mma = [&](const Regs& rg) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int e = 0; e < W; ++e)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            gacc[e][nb] = M::run(run_elem(rg.xa[u][s], e), rg.ra[u][nb][s / E][s % E], gacc[e][nb]);
  };
  // Explicit waits leave the group just issued in flight (the compiler, left to itself,
  // waits for every load before the first MFMA of the rotated loop).
  constexpr int GL = U * (4 + NB * RB);            // loads per group
  static_assert(GL < 64, "vmcnt range");
  // Groups are taken in pairs; with an odd count the last pair's second group is one of
  // zeros, whose products add nothing.
  Regs r0, r1;
  load(ngroups - 1, r0);
  for (int64_t k = ngroups - 1; k >= 0; k -= 2) {
    load(k - 1, r1);
    __builtin_amdgcn_s_waitcnt(wait_vm(GL));
    mma(r0);
    load(k - 2, r0);
    __builtin_amdgcn_s_waitcnt(wait_vm(GL));
    mma(r1);
  }

  // row r of accumulator e is column j0 + W row + e
  auto column = [&](int e, int r) { return j0 + M::row(r, g) * W + e; };
  if (gridDim.y > 1) {
    T* gp = static_cast<T*>(a.gpart) + (int64_t)blockIdx.y * a.gstride;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int e = 0; e < W; ++e) {
          const int j = column(e, r), k = nb * 16 + c;
          if (j < p && k < K) gp[(int64_t)j * K + k] = gacc[e][nb][r];
        }
    return;
  }

  // epilogue on this lane's elements (same arithmetic as the row-tile epilogue); the
  // position and momentum are read only now, after the stream
  T* Bv = static_cast<T*>(a.B);
  T* Ev = static_cast<T*>(a.eta);
  T* Gv = static_cast<T*>(a.G);
  double pr = 0.0, ke = 0.0;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int el = 0; el < W; ++el) {
        const int j = column(el, r), k = nb * 16 + c;
        if (j >= p || k >= K) continue;
        const int64_t e = (int64_t)j * K + k;
        const bool pinned = a.pin && k == K - 1;
        const T bt = Bv[e];
        const double b = (double)bt;
        const T gt = pinned ? T(0) : (T)((double)gacc[el][nb][r] + prior_grad(b, a.prior, a.scale));
        Gv[e] = gt;
        pr += pinned ? 0.0 : prior_logd(b, a.prior, a.scale);
        if (a.mode != 0) {
          const T h = (T)a.h;
          T ev = Ev[e] + h * gt;                               // closing half kick
          if (a.mode == 1) {
            ev = ev + h * gt;                                  // opening half kick
            Bv[e] = pinned ? T(0) : bt + (T)a.eps * ev;        // position step
          } else {
            ke += 0.5 * (double)ev * (double)ev;
          }
          Ev[e] = ev;
        }
      }
  pr = wave_sum(pr);
  ke = wave_sum(ke);
  if (lane == 0) { sh4[0][w] = pr; sh4[1][w] = ke; }
  __syncthreads();
  if (tid == 0) {
    a.ppart[blockIdx.x] = ((sh4[0][0] + sh4[0][1]) + sh4[0][2]) + sh4[0][3];
    if (a.mode == 2) a.kpart[blockIdx.x] = ((sh4[1][0] + sh4[1][1]) + sh4[1][2]) + sh4[1][3];
  }
}

}  // namespace

template <typename T>
int wide_chunk_cols() { return wide_chunk<T>(); }
// Workgroups of the column-owner gradient for p columns, by 16-byte loads or narrow.
int wide_grad_groups(int64_t p, bool f64, bool narrow) {
  const int64_t cols = (int64_t)kWideWaves * 16 * (narrow ? 1 : f64 ? 2 : 4);
  return (int)((p + cols - 1) / cols);
}
// Row slices wanted for p columns: about 512 / g with g the workgroups that hold at most 4 (2 in
// float64, fewer with more class blocks) blocks of 16 columns per wave, in whole rounds of 256
// from 256 on and 256 while that leaves a wave two blocks. More slices made some shapes 4-8%
// faster and others as much slower.
int wide_row_slices(int64_t p, int nb, bool f64) {
  const int64_t nblk = (p + 15) / 16;
  const int cb = f64 ? (nb == 1 ? 2 : 1) : (nb == 1 ? 4 : nb == 2 ? 2 : 1);
  int64_t g = (nblk + kWideWaves * cb - 1) / (kWideWaves * cb);
  if (g >= 256) g = (g + 255) / 256 * 256;
  else if (nblk >= (int64_t)kWideWaves * 256 * 2) g = 256;
  return g < 512 ? (int)((512 + g - 1) / g) : 1;
}
// Logits workgroups a compute unit holds at once (registers: 163, 235 and 375 per lane with 1, 2
// and 4 class blocks).
int wide_logits_resident(int nb) { return nb == 1 ? 3 : nb == 2 ? 2 : 1; }

template <typename T>
hipError_t launch_wide(const WideArgs& a, int nb, int logits_tiles_y, int softmax_wg, int grad_wg,
                       bool narrow, hipStream_t s) {
  const dim3 lg(a.nchunk, logits_tiles_y);
  const dim3 gg(grad_wg, a.nsplit);
#define HMC_WIDE(NB_)                                                                       \
  if (nb == NB_) {                                                                          \
    hipLaunchKernelGGL((wide_logits<T, NB_>), lg, dim3(kWideWaves * 64), 0, s, a);          \
    hipLaunchKernelGGL((wide_softmax<T, NB_>), dim3(softmax_wg), dim3(256), 0, s, a);       \
    if (narrow) hipLaunchKernelGGL((wide_grad<T, NB_, 1>), gg, dim3(kWideWaves * 64), 0, s, a); \
    else hipLaunchKernelGGL((wide_grad<T, NB_, 16 / (int)sizeof(T)>), gg, dim3(kWideWaves * 64), 0, s, a); \
    return hipGetLastError();                                                               \
  }
  HMC_WIDE(1) HMC_WIDE(2) HMC_WIDE(4)
#undef HMC_WIDE
  return hipErrorInvalidValue;
}

template int wide_chunk_cols<float>();
template int wide_chunk_cols<double>();
template hipError_t launch_wide<float>(const WideArgs&, int, int, int, int, bool, hipStream_t);
template hipError_t launch_wide<double>(const WideArgs&, int, int, int, int, bool, hipStream_t);

}  // namespace hmcx
