// Fused log-posterior + gradient pass for one free coefficient column: the Poisson and probit
// links, and the two-class logit with its last class pinned.
//
// With one column the contractions are two multiply-adds per element of X, and reading X (once)
// is all that matters; the row tile's matrix instructions would spend 15 of 16 output columns
// and its barriers on them. Here half a wave owns a row, a lane 16 columns of each 512: the row
// goes from memory to registers, is multiplied with the coefficients, the lanes' sums are
// exchanged within the wave, and the row is added into the gradient held in registers, without a
// barrier until the waves of the workgroup add up their gradients at the end. Two pairs of rows
// are in flight per wave while one is used. Poisson, FP32, n = 20000, p = 1000 (80 MB): 16.5 us,
// 4.9 TB/s, of which about 5 us are the launch, the first load and the last sums, against the row
// tile's 21.4; n = 200000, p = 256, whole gradient: 37 us against 56.
//
// In float32 the logit's order of summation is the row tile's: lane l of the half adds columns t,
// 4 + t, 8 + t, 12 + t (t = 0 .. 3) of block l, then of block l + 32, by fused multiply-adds; lanes
// w and w + 16 are added, then w = 0 .. 15 in turn. log K thus keeps its bits but for the order of
// the float64 sum over rows. So a lane loads whole blocks, 64 bytes in four loads; in float64,
// where any order will do, neighbouring lanes load neighbouring pieces. (The float64 probit link's
// function leaves 40 bytes of a lane's state in scratch.)
#include <math.h>

#include "device_common.h"

namespace hmcx {
namespace {

using namespace dev;

constexpr int kColumnWaves = 8;

// MBL: 16-column blocks per lane. LINK as in FusedArgs (0: two classes, the last pinned).
template <typename T, int MBL, int LINK, int AUX>
__global__ __launch_bounds__(64 * kColumnWaves, 2) void column_pass(FusedArgs a) {
  constexpr int E = 16 / sizeof(T);                // elements per 16-byte load
  constexpr int PC = 16 / E;                       // loads per block
  constexpr bool ORDER = sizeof(T) == 4;           // the row tile's order of summation
  constexpr int COLS = 512 * MBL;                  // 64 kColumnWaves MBL
  typedef T vec_t __attribute__((ext_vector_type(E)));
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ __align__(16) T zx[kColumnWaves][64];
  __shared__ double lsum[kColumnWaves];
  T* gx = reinterpret_cast<T*>(smem);              // [2 kColumnWaves][COLS] gradients
  T* bs = gx + 2 * kColumnWaves * COLS;            // [COLS] coefficients
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, hl = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int p = a.p, K = a.K;
  const int64_t n = a.n, ldx = a.ldx;
  const T* X = static_cast<const T*>(a.X);
  const T* B = static_cast<const T*>(a.B);
  if (a.ticket && blockIdx.x == 0 && tid == 0) *a.ticket = 0;

  T gv[MBL][16];
#pragma unroll
  for (int m = 0; m < MBL; ++m)
#pragma unroll
    for (int e = 0; e < 16; ++e) gv[m][e] = T(0);
  // Load u of block group m starts at this column.
  auto column = [&](int m, int u) { return ORDER ? 16 * (hl + 32 * m) + u * E : 512 * m + (32 * u + hl) * E; };
  // The one load that reaches past column p, if any.
  const bool ragged = p % E != 0;
  const int rm = p / 512, ru = ORDER ? p % 16 / E : p % 512 / (32 * E);
  const bool mine = hl == (ORDER ? p / 16 % 32 : p / E % 32);
  double lacc = 0.0;

  const int64_t pairs = (n + 1) / 2, step = (int64_t)gridDim.x * kColumnWaves;
  struct Rows { vec_t v[MBL][PC]; int y; };
  // Rows 2 q and 2 q + 1. A load at or past column p, and a pair past the last, goes past the
  // resource's end: zeros, no traffic.
  auto load = [&](int64_t q, Rows& r) {
    const bool real = q < pairs;
    const int64_t i0 = real ? 2 * q : 0;
    const __amdgpu_buffer_rsrc_t xr =
        make_rsrc(X + i0 * ldx, real ? (uint64_t)((i0 + 1 < n ? ldx : 0) + p) * sizeof(T) : 0);
    const __amdgpu_buffer_rsrc_t yr = make_rsrc(a.y + i0, real ? (i0 + 1 < n ? 8 : 4) : 0);
#pragma unroll
    for (int m = 0; m < MBL; ++m)
#pragma unroll
      for (int u = 0; u < PC; ++u) {
        const int col = column(m, u);
        r.v[m][u] = __builtin_bit_cast(vec_t, __builtin_amdgcn_raw_buffer_load_b128(
            xr, col < p ? (int)((half * ldx + col) * sizeof(T)) : (int)0xFFFFFFF0u, 0, AUX));
      }
    r.y = __builtin_amdgcn_raw_buffer_load_b32(yr, half * 4, 0, 0);
  };
  auto use = [&](int64_t q, Rows& r) {
    if (ragged) {
#pragma unroll
      for (int m = 0; m < MBL; ++m)
#pragma unroll
        for (int u = 0; u < PC; ++u)
          if (m == rm && u == ru) {
#pragma unroll
            for (int e = 0; e < E; ++e) r.v[m][u][e] = mine && e >= p % E ? T(0) : r.v[m][u][e];
          }
    }
    T z = T(0), z0 = T(0);                         // z0: the pinned class's, formed only if needed
#pragma unroll
    for (int m = 0; m < MBL; ++m) {
      vec_t b[PC];
#pragma unroll
      for (int u = 0; u < PC; ++u) b[u] = *reinterpret_cast<const vec_t*>(bs + ((m * PC + u) * 32 + hl) * E);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int e = 4 * c + t;
          z = fma(r.v[m][e / E][e % E], b[e / E][e % E], z);
        }
    }
    if constexpr (ORDER) {
      __builtin_amdgcn_wave_barrier();             // the previous pair's sums are read
      zx[w][lane] = z;
      __builtin_amdgcn_wave_barrier();
      vec_t zs[32 / E];
#pragma unroll
      for (int i = 0; i < 32 / E; ++i) zs[i] = *reinterpret_cast<const vec_t*>(&zx[w][32 * half + i * E]);
      z = zs[0][0] + zs[16 / E][0];
#pragma unroll
      for (int i = 1; i < 16; ++i) z += zs[i / E][i % E] + zs[(16 + i) / E][i % E];
    } else {
#pragma unroll
      for (int t = 16; t >= 1; t >>= 1) z += __shfl_xor(z, t, 32);
    }
    const bool valid = 2 * q + half < n;
    T res;
    double l;
    if constexpr (LINK == 1) {
      const T mu = dev_exp(z);
      res = T(r.y) - mu;
      l = (double)r.y * (double)z - (double)mu;
    } else if constexpr (LINK == 2) {
      const T s = r.y == 1 ? T(1) : T(-1);
      T ratio;
      probit_row(valid ? s * z : T(0), ratio, l);
      res = s * ratio;
    } else {
      // x * 0 summed is the pinned logit: NaN in a row that holds an infinity or a NaN, which
      // also leaves z infinite or NaN
      if (__builtin_amdgcn_ballot_w64(!(fabs(z) <= (T)INFINITY) || fabs(z) == (T)INFINITY)) {
        T bad = T(0);
#pragma unroll
        for (int m = 0; m < MBL; ++m)
#pragma unroll
          for (int e = 0; e < 16; ++e) bad = fma(r.v[m][e / E][e % E], T(0), bad);
#pragma unroll
        for (int s = 16; s >= 1; s >>= 1) bad += __shfl_xor(bad, s, 32);
        z0 = bad;
      }
      const T mx = fmax(fmax((T)-INFINITY, z), z0);
      const T ez = dev_exp(z - mx), e0 = dev_exp(z0 - mx);
      const T se = ez + e0;
      const T inv = dev_rcp(se), lse_shift = dev_log(se);
      res = (r.y == 0 ? T(1) : T(0)) - ez * inv;
      // as on the row tile: no term for a label outside the 16 padded classes
      l = (unsigned)r.y < 16u ? (double)(((r.y == 0 ? z : z0) - mx) - lse_shift) : 0.0;
    }
    if (!valid) res = T(0);
    lacc += valid && hl == 0 ? l : 0.0;
#pragma unroll
    for (int m = 0; m < MBL; ++m)
#pragma unroll
      for (int e = 0; e < 16; ++e) gv[m][e] = fma(r.v[m][e / E][e % E], res, gv[m][e]);
  };
  T bj[MBL];
#pragma unroll
  for (int m = 0; m < MBL; ++m) bj[m] = tid + 512 * m < p ? B[(int64_t)(tid + 512 * m) * K] : T(0);
  // Two pairs in flight while one is used; one in float64, whose registers hold no more. The first
  // are under way while the coefficients are staged.
  int64_t q = (int64_t)blockIdx.x * kColumnWaves + w;
  Rows r0, r1, r2;
  load(q, r0);
  if constexpr (sizeof(T) == 4) load(q + step, r1);
  // The coefficients, a lane's 16-byte pieces next to its neighbours': no bank conflicts.
#pragma unroll
  for (int m = 0; m < MBL; ++m) {
    const int j = tid + 512 * m, b = j / 16, u = j % 16 / E;
    bs[ORDER ? ((m * PC + u) * 32 + b % 32) * E + j % E : j] = bj[m];
  }
  __syncthreads();
  if constexpr (sizeof(T) == 4) {
    while (q < pairs) {
      load(q + 2 * step, r2);
      use(q, r0);
      if ((q += step) >= pairs) break;
      load(q + 2 * step, r0);
      use(q, r1);
      if ((q += step) >= pairs) break;
      load(q + 2 * step, r1);
      use(q, r2);
      q += step;
    }
  } else {
    while (q < pairs) {
      load(q + step, r1);
      use(q, r0);
      if ((q += step) >= pairs) break;
      load(q + step, r0);
      use(q, r1);
      q += step;
    }
  }

  // the workgroup's partial: halves and waves added in order
  T* gh = gx + (2 * w + half) * COLS;
#pragma unroll
  for (int m = 0; m < MBL; ++m)
#pragma unroll
    for (int e = 0; e < 16; e += E)
      *reinterpret_cast<vec_t*>(gh + column(m, e / E)) = *reinterpret_cast<const vec_t*>(&gv[m][e]);
  lacc = wave_sum(lacc);
  if (lane == 0) lsum[w] = lacc;
  __syncthreads();
  T* gp = static_cast<T*>(a.gpart) + (int64_t)blockIdx.x * a.gstride;
  for (int j = tid; j < p; j += 64 * kColumnWaves) {
    T s = gx[j];
#pragma unroll
    for (int i = 1; i < 2 * kColumnWaves; ++i) s += gx[i * COLS + j];
    gp[(int64_t)j * K] = s;
    if (K == 2) gp[(int64_t)j * K + 1] = T(0);     // the pinned column
  }
  if (tid == 0) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kColumnWaves; ++i) s += lsum[i];
    a.lpart[blockIdx.x] = s;
  }
}

template <typename T, int MBL, int LINK, int AUX>
hipError_t launch_variant(const FusedArgs& a, int nwg, hipStream_t s) {
  constexpr int lds = (2 * kColumnWaves + 1) * 512 * MBL * (int)sizeof(T);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&column_pass<T, MBL, LINK, AUX>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((column_pass<T, MBL, LINK, AUX>), dim3(nwg), dim3(64 * kColumnWaves), lds, s, a);
  return hipGetLastError();
}

// Non-temporal loads gain where a load instruction takes whole lines (float64) and a row is many
// lines long: n = 200000, p = 512: 132 us against 149; p = 200 (a million rows): 261 against 282;
// p = 100, where the lines that two loads share count for more: 53 against 44. The float32 layout
// takes each line in four loads, which must find it in the cache (143 us became 224).
constexpr int kStreamCols = 192, kNonTemporal = 2;

template <typename T, int MBL, int LINK>
hipError_t launch_one(const FusedArgs& a, int nwg, hipStream_t s) {
  if constexpr (sizeof(T) == 8 && LINK == 2) {    // more than 256 columns (column_fits)
    return launch_variant<T, MBL, LINK, kNonTemporal>(a, nwg, s);
  } else {
    if constexpr (sizeof(T) == 8) {
      if (a.p >= kStreamCols) return launch_variant<T, MBL, LINK, kNonTemporal>(a, nwg, s);
    }
    return launch_variant<T, MBL, LINK, 0>(a, nwg, s);
  }
}

}  // namespace

// One free column, and columns that the lanes of half a wave hold: as many as the row tile takes.
// The row tile keeps (us here against there)
//  - small problems, whose waves have less to set up there: float32, n = 5000, p = 32: 10.0 against 9.7
//    (n = 20000: 11.3 against 12.0; n = 50, p = 192: 9.0 against 9.5); float64, n = 27935, p = 51, K = 2:
//    22.1 against 20.4 (n = 20000, p = 128: 17.0 against 17.9);
//  - rows of a few floats, of which a wave here takes two and a tile there sixteen, below the sizes
//    where that tells: Poisson, five updates, p = 3: n = 15000 51.5 against 48.1, n = 60000 83.1 against
//    80.9, n = 120000 124 against 127; p = 6: n = 10000 49.6 against 47.0, n = 15000, p = 5: 50.5 against 51.7;
//  - float64 probit problems of few columns: its link function, here evaluated for two rows per wave,
//    there for four, is then what takes the time (n = 200000, p = 128: 92 against 84; p = 384: 123
//    against 145);
//  - float64 two-class problems of up to 128 columns in odd number without row padding, whose rows
//    start off 16-byte pieces here while the tile there needs no mask: n = 92307, p = 65: 44.4 against
//    41.4 (with a padded row 43.8 against 46.7; p = 151: 57.9 against 72.6).
bool column_fits(int64_t n, int64_t p, int K, bool pin, bool f64, int link, int64_t ldx) {
  if ((pin ? K - 1 : K) != 1) return false;
  if (!f64) return p <= 1024 && (p > 128 || n >= (p < 4 ? 65536 : p < 16 ? 16384 : 8192));
  if (link == 0 && p <= 128 && p % 2 && ldx == p) return false;
  return p <= 512 && n * p >= (p >= 256 ? 1 << 20 : 1 << 21) && (link != 2 || p > 256);
}
// A workgroup per compute unit, each wave with a pair of rows at least.
int column_workgroups(int64_t n) {
  const int64_t g = ((n + 1) / 2 + kColumnWaves - 1) / kColumnWaves;
  return (int)(g < 256 ? g : 256);
}

template <typename T>
hipError_t launch_column(const FusedArgs& a, int nwg, hipStream_t s) {
#define HMC_COLUMN(MBL_) \
  a.link == 1 ? launch_one<T, MBL_, 1>(a, nwg, s) : a.link == 2 ? launch_one<T, MBL_, 2>(a, nwg, s) \
                                                                : launch_one<T, MBL_, 0>(a, nwg, s)
  if constexpr (sizeof(T) == 4) {
    if (a.p > 512) return HMC_COLUMN(2);
  }
  return HMC_COLUMN(1);
#undef HMC_COLUMN
}

template hipError_t launch_column<float>(const FusedArgs&, int, hipStream_t);
template hipError_t launch_column<double>(const FusedArgs&, int, hipStream_t);

}  // namespace hmcx
