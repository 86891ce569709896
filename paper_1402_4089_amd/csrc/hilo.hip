// Split-precision form of the gradient pass. X is stored as two bfloat16 planes
// (hi = bf16(X), lo = bf16(X - hi)); the FP32 operands it meets (the coefficients B and
// the residuals R = Y - P) are split the same way on the fly, and each contraction sums
// the three products hi*hi + hi*lo + lo*hi on the BF16 matrix cores (v_mfma 16x16x32)
// with FP32 accumulation. Softmax statistics (log-sum-exp, the log-likelihood) are
// formed in FP64.
//
// The per-class gradient of this form does not fit one compute unit (p*K FP32
// accumulators exceed its register file), so the pass runs as two kernels: row blocks
// compute logits, softmax and the packed residual; column blocks then accumulate
// X^T R over a slice of rows each, and the shared epilogue sums the slices.
#include <math.h>

#include <algorithm>
#include <utility>

#include "device_common.h"

namespace hmcx {
namespace {

using namespace dev;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// bfloat16 of a double, rounded once to nearest even: 8 significant bits, the exponent
// range of binary32 (subnormals spaced 2^-133), +-inf past the largest finite value. The
// double goes through binary32 rounded to odd: of the two neighbours of an inexact value the
// one with an odd last bit, so that rounding its 24 bits to 8 rounds the value itself once.
__device__ __forceinline__ u16 bf16_from_f64(double x) {
  if (x != x) return (u16)(((uint64_t)__double_as_longlong(x) >> 48 & 0x8000u) | 0x7FC0u);
  float f = (float)x;
  const double d = (double)f;
  uint32_t u = __float_as_uint(f);
  // d is off by less than one step: the odd neighbour lies on the side of x (past the largest
  // finite binary32, d = inf: one step down, which rounds to inf again)
  if (d != x && !(u & 1u)) u += (fabs(x) > fabs(d)) ? 1u : -1u;
  return bf16_from_f32(__uint_as_float(u));
}

__device__ __forceinline__ uint32_t pack2(u16 a, u16 b) { return (uint32_t)a | ((uint32_t)b << 16); }

__device__ __forceinline__ bf16x8 as_frag(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Two transposing reads of 4 rows x 16 columns (per 16-lane group) as the 8 elements of an operand.
__device__ __forceinline__ u32x4 tr_pair(const u16* a, const u16* b) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const uint2 u = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)a));
  const uint2 v = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)b));
  return u32x4{u.x, u.y, v.x, v.y};
}

__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------------------
// Encoding of X: one thread per 8 output columns of a row; columns [p, ldo) are zeroed. Memory
// bounds it: sizeof(Tin) bytes read and 2 or 4 written per element. A workgroup takes `rows` rows of
// `span` groups of 8 columns, a thread UNROLL groups at a time, all of whose loads are issued before
// the first conversion. The differences x - hi are exact in the type of X (hi holds the leading bits
// of x), so FP32 X is encoded in FP32: both planes have the bits of the conversion through float64, a
// NaN's sign and quiet bit included. Measured, n = 50000, p = 4096, FP32 to both planes: 297 us (5.5
// TB/s; a device copy of that size reaches 4.8), against 596 us with one group per thread in flight,
// element loads, a 64-bit division per group and integer rounding of doubles.
//
// A workgroup has kSplitGroups groups of whole rows, two rounds of four per thread, where that makes
// kSplitWorkgroups of them or more. A smaller X takes a round's latency, not the rate: fewer groups
// per workgroup then, down to one per thread, and pieces of the rows; so do fewer than 8 columns,
// whose groups are padding but one per row (us with one group per thread against two rounds of
// four: n = 3027, p = 366, FP64: 4.9, 13.4; n = 17041, p = 1, FP32: 3.2, 8.6).
constexpr int kSplitUnroll = 4, kSplitGroups = 256 * kSplitUnroll * 2, kSplitWorkgroups = 2048;
constexpr int64_t kSplitSpan = 1 << 20;          // column groups of one grid row at most

__device__ __forceinline__ void split_one(double x, u16& h, u16& l) {
  h = bf16_from_f64(x);
  l = bf16_from_f64(x - (double)f32_from_bf16(h));
}
__device__ __forceinline__ u16 bf16_quiet(float x) {
  return x != x ? (u16)((__float_as_uint(x) >> 16 & 0x8000u) | 0x7FC0u) : bf16_from_f32(x);
}
__device__ __forceinline__ void split_one(float x, u16& h, u16& l) {
  h = bf16_quiet(x);
  l = bf16_quiet(x - f32_from_bf16(h));
}

template <typename Tin, int UNROLL>
__global__ __launch_bounds__(256) void split_kernel(const Tin* __restrict__ X, int64_t ldx,
                                                    int64_t n, int64_t p, u16* __restrict__ hi,
                                                    u16* __restrict__ lo, int64_t ldo, uint32_t rows,
                                                    int64_t span) {
  struct alignas(sizeof(Tin)) Run { Tin v[8]; };      // 8 elements at any element address
  const int64_t r0 = (int64_t)blockIdx.x * rows;
  const int64_t g0 = (int64_t)blockIdx.y * span;      // first column group of this workgroup
  const uint32_t gpr = (uint32_t)(ldo / 8 - g0 < span ? ldo / 8 - g0 : span);
  const uint32_t total = (uint32_t)(n - r0 < rows ? n - r0 : rows) * gpr;
  for (uint32_t t0 = threadIdx.x; t0 < total; t0 += 256 * UNROLL) {
    Run x[UNROLL];
    int64_t row[UNROLL], c0[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const uint32_t t = t0 + 256 * u, i = t / gpr;
      row[u] = r0 + i;
      c0[u] = (g0 + (t - i * gpr)) * 8;
      if (t < total && c0[u] + 8 <= p) {
        x[u] = *reinterpret_cast<const Run*>(X + row[u] * ldx + c0[u]);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          x[u].v[j] = (t < total && c0[u] + j < p) ? X[row[u] * ldx + c0[u] + j] : Tin(0);
      }
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      if (t0 + 256 * u >= total) break;
      u16 h[8], l[8];
      if (UNROLL > 1 || p >= 8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) split_one(x[u].v[j], h[j], l[j]);
      } else {                                        // all else is padding
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          h[j] = l[j] = 0;
          if (j < p) split_one(x[u].v[j], h[j], l[j]);
        }
      }
      const int64_t o = row[u] * ldo + c0[u];
      *reinterpret_cast<u32x4*>(hi + o) =
          u32x4{pack2(h[0], h[1]), pack2(h[2], h[3]), pack2(h[4], h[5]), pack2(h[6], h[7])};
      if (lo)
        *reinterpret_cast<u32x4*>(lo + o) =
            u32x4{pack2(l[0], l[1]), pack2(l[2], l[3]), pack2(l[4], l[5]), pack2(l[6], l[7])};
    }
  }
}

// ---------------------------------------------------------------------------------------
// One problem's operands for the split-precision bodies below. Class blocks: the padded
// class axis is NB blocks of 16, in softmax groups of GROUP blocks. With GROUP == NB the
// blocks are one problem's K <= 16 NB classes (one softmax per row); with GROUP < NB each
// group is a separate chain of the same problem with K <= 16 GROUP classes (NB / GROUP
// chains share every pass over X, one softmax per row and chain). A chain's state,
// gradient and partials are chain-major [chain][p][K].
struct Job {
  const u16* Xhi;
  const u16* Xlo;
  int64_t ldx;
  const int32_t* y;
  int64_t n;
  int p, K;
  const float* B;
  u16* Bpk;
  u16* Rpk;
  int pin;                 // 1: column K-1 of B is packed as zero (beta_K = 0)
};

// Cache policy of the loads of X (the aux operand of a buffer load): some row slices (as many
// as fit the memory-side cache, spread evenly over X so that its bandwidth and the memory's
// add up) are read with the default policy and found there again by the other pass, the rest
// with the non-temporal hint, which streams faster and leaves the cached part alone. The X
// loads of both passes use whole 128-byte lines.
constexpr int kKeep = 0, kStream = 2;
__device__ __forceinline__ bool hot_slice(int64_t s, int share) {
  return (int)((uint32_t)s * (uint32_t)share & 0xFFFFu) < share;
}

// B -> packed hi/lo operand in the lane order of the MFMA B input: fragment (k-step s,
// class block nb, plane) holds, for lane l, the 8 values B[32 s + 8 (l / 16) + j][class
// 16 nb + l % 16 of the block's group], j = 0..7. Padding rows and classes are zero.
template <int NB, int GROUP>
__device__ __forceinline__ void pack_b_body(const Job& j, int64_t t) {
  const int lane = (int)(t & 63);
  const int nb = (int)((t >> 6) % NB);
  const int ks = (int)(t / (64 * NB));
  const int kk = 16 * (nb % GROUP) + (lane & 15);
  const int pb = 32 * ks + 8 * (lane >> 4);
  const float* B = j.B + (int64_t)(nb / GROUP) * j.p * j.K;
  const int kmax = j.pin ? j.K - 1 : j.K;
  u16 h[8], l[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float v = (pb + e < j.p && kk < kmax) ? B[(int64_t)(pb + e) * j.K + kk] : 0.0f;
    h[e] = bf16_from_f32(v);
    l[e] = bf16_from_f32(v - f32_from_bf16(h[e]));
  }
  u16* dst = j.Bpk + packed_b_index(NB, nb, pb, lane & 15);
  *reinterpret_cast<u32x4*>(dst) = u32x4{pack2(h[0], h[1]), pack2(h[2], h[3]), pack2(h[4], h[5]), pack2(h[6], h[7])};
  *reinterpret_cast<u32x4*>(dst + 512) = u32x4{pack2(l[0], l[1]), pack2(l[2], l[3]), pack2(l[4], l[5]), pack2(l[6], l[7])};
}

// Logits, softmax and packed residuals of row block rb (kHiloRows rows); every thread
// of the workgroup takes part (barriers inside).
//
// Reading X bounds this: 2 or 4 bytes per element once, the matrix cores are busy a quarter
// of that time. Wave w owns kHiloMB 16-row M blocks and all 16*NB padded classes. The MFMA A
// operand wants, of each 32-column k step, 8 consecutive columns of row l % 16 in lane l, but
// loads of that shape (16 rows x 64 bytes per instruction, the four lanes of a row 16 lanes
// apart) stream at 4.2 TB/s (n = 200000, p = 4096). X is therefore read in chunks of 64
// columns, 8 rows x 128 bytes (whole lines) per instruction, kXDepth chunks ahead in registers, and each chunk goes through a piece of LDS that only its wave touches:
// stored by rows, read back as operands, the 16-byte pieces of a row XOR-ed with (row / 2) % 8
// so that both accesses are free of bank conflicts. The packed B operand, shared by all
// waves, is staged in LDS (`bs`, two buffers of kBSteps k steps) one chunk ahead. After the k
// loop, lane l holds logits of rows 4 (l / 16) + i (i < 4) for class 16 nb + l % 16, so every
// row is spread over one 16-lane DPP row: max and sum are DPP reductions (across the GROUP
// blocks of a softmax group in-lane). The residual R = onehot(y) - P is split into bf16
// hi/lo and stored in the B-input lane order of the gradient kernel. lacc[group] gains
// this wave's log-likelihood terms (in the lane holding each row's label).
//
// LDS per workgroup: X 16 KB a plane and B 32 KB (16 KB for one class block), so that two
// workgroups share a compute unit; the X registers of kXDepth chunks are 64 either way.
template <int NB> constexpr int kBSteps = NB == 4 ? 2 : 4;         // k steps of B per LDS buffer
template <bool LO> constexpr int kXDepth = LO ? 2 : 4;             // 64-column chunks of X in flight
template <int NB> constexpr int bchunk_elems() { return kBSteps<NB> * NB * 1024; }
template <int NB, bool LO> constexpr int logits_lds_elems() {
  return 2 * bchunk_elems<NB>() + (LO ? 2 : 1) * kHiloRows * 64;
}

// lse[v] = zmx[v] + the log held by the lane of the row that has sum v.
template <int F, int... V>
__device__ __forceinline__ void read_logs(double lg, const float (&zmx)[F], double (&lse)[F],
                                          std::integer_sequence<int, V...>) {
  ((lse[V] = (double)zmx[V] + dpp<kRowBcast + row_sum_lane(V)>(lg)), ...);
}

// Softmax over the K valid classes of each row and group of row block rb, FP64 statistics,
// and the packed residuals. The sums of exponentials of a lane's 4 rows x NG groups are formed
// one per lane (row_sums), where the FP64 log is taken, and read back from that lane by the
// others of the row. lacc[group] gains this wave's log-likelihood terms (in the label's lane).
// Vector work bounds it (no other kernel of the pass overlaps it within the workgroup): per
// pair of elements two exponentials each, three FP64 operations and the two packed
// conversions of the residual's planes.
template <int NB, int GROUP>
__device__ __forceinline__ void softmax_residuals(const Job& j, int64_t rb,
                                                  const f32x4 (&acc)[kHiloMB][NB],
                                                  const int (&ylab)[kHiloMB][4],
                                                  double (&lacc)[NB / GROUP]) {
  constexpr int NG = NB / GROUP;
  constexpr int MB = kHiloMB;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int m = lane & 15, g = lane >> 4;
  const int64_t n = j.n;
  const int K = j.K;
  const int64_t r0 = rb * kHiloRows + (int64_t)w * 16 * MB;
  constexpr int F = 4 * NG;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int64_t rblk = r0 / 32 + mb / 2;     // 32-row block of the gradient kernel
    float zmx[F];
    double ssum[16];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        float zmax = -INFINITY;
#pragma unroll
        for (int b = 0; b < GROUP; ++b)
          if (16 * b + m < K) zmax = fmaxf(zmax, acc[mb][q * GROUP + b][i]);
        zmax = max16(zmax);
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < GROUP; ++b)
          if (16 * b + m < K) s += (double)dev_exp(acc[mb][q * GROUP + b][i] - zmax);
        zmx[i * NG + q] = zmax;
        ssum[i * NG + q] = s;
      }
    const double lg = log(row_sums<F>(ssum));
    double lse[F];
    read_logs<F>(lg, zmx, lse, std::make_integer_sequence<int, F>{});
    uint32_t rh[NB][2], rl[NB][2];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int q = nb / GROUP, kk = 16 * (nb % GROUP) + m;
      float r[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool valid = r0 + 16 * mb + 4 * g + i < n && kk < K;
        const bool hit = valid && kk == ylab[mb][i];
        const double zl = (double)acc[mb][nb][i] - lse[i * NG + q];   // log softmax
        lacc[q] += hit ? zl : 0.0;                                    // the label's lane only
        r[i] = valid ? (hit ? 1.0f : 0.0f) - dev_exp((float)zl) : 0.0f;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        rh[nb][h] = bf16x2_from_f32(r[2 * h], r[2 * h + 1]);
        rl[nb][h] = bf16x2_from_f32(r[2 * h] - __uint_as_float(rh[nb][h] << 16),
                                    r[2 * h + 1] - __uint_as_float(rh[nb][h] & 0xFFFF0000u));
      }
    }
    // rows 16 (mb % 2) + 4 g + i of this 32-row block sit in lane 16 (2 (mb % 2) + g / 2)
    // + m, elements 4 (g % 2) + i, of the gradient kernel's fragments
    const int L = 16 * (2 * (mb & 1) + (g >> 1)) + m;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      u16* f = j.Rpk + (rblk * NB + nb) * 2 * 512 + L * 8 + 4 * (g & 1);
      *reinterpret_cast<uint2*>(f) = uint2{rh[nb][0], rh[nb][1]};
      *reinterpret_cast<uint2*>(f + 512) = uint2{rl[nb][0], rl[nb][1]};
    }
  }
}

template <int NB, int GROUP, bool LO, int AUX>
__device__ __forceinline__ void logits_rows(const Job& j, int64_t rb, double (&lacc)[NB / GROUP],
                                            u16* __restrict__ bs) {
  constexpr int PL = LO ? 2 : 1;
  constexpr int BST = kBSteps<NB>, XD = kXDepth<LO>;
  constexpr int CH = bchunk_elems<NB>();         // u16 per B chunk (hi and lo fragments)
  constexpr int PER = CH / 8 / (kHiloWaves * 64);   // 16-byte pieces per thread per chunk
  static_assert(CH / 8 % (kHiloWaves * 64) == 0, "a B chunk is a whole number of 16-byte pieces per thread");
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int64_t n = j.n;
  const int p = j.p;
  const int nks = (p + 31) / 32, nxc = (nks + 1) / 2;   // k steps, 64-column chunks
  constexpr int MB = kHiloMB;
  f32x4 acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // X comes from branch-free buffer loads whose resource starts at the row block and ends with
  // it or at row n, so rows past n read as zero. A block spans less than 2^31 bytes (ldx < 2^23),
  // so the offset 0xFFFFFFF0 of a piece past column p lies beyond it however large X is: with all
  // of X in the resource that offset fell inside a plane of more than 4 GiB, on any element or
  // row padding there, whose NaN times a zero coefficient reached the logits. Instruction i loads
  // rows 8 i + lane / 8 of the wave's 32, 16-byte piece lane % 8 of the chunk.
  const int64_t rbase = rb * kHiloRows;
  const int64_t brows = n - rbase < kHiloRows ? n - rbase : kHiloRows;
  const uint64_t rem = (uint64_t)brows * j.ldx * 2;
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(j.Xhi + rbase * j.ldx, rem);
  const __amdgpu_buffer_rsrc_t rl = make_rsrc(LO ? j.Xlo + rbase * j.ldx : j.Xhi, LO ? rem : 0);
  const int piece = lane & 7;
  uint32_t xoff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    xoff[i] = (uint32_t)(((int64_t)(w * 32 + 8 * i + (lane >> 3)) * j.ldx + 8 * piece) * 2);
  // labels of this lane's rows, loaded now so their latency hides behind the k loop
  // (rows past n read as zero and are not used)
  const __amdgpu_buffer_rsrc_t yres = make_rsrc(j.y + rbase, (uint64_t)(n - rbase) * 4);
  int ylab[MB][4];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      ylab[mb][i] = __builtin_amdgcn_raw_buffer_load_b32(
          yres, (int)((w * 16 * MB + 16 * mb + 4 * g + i) * 4), 0, 0);
  const int nch = (nks + BST - 1) / BST;
  const int64_t bp_total = (int64_t)nks * NB * 1024;
  u32x4 bst[PER];
  // every load below is issued unconditionally: buffer loads past a resource's end read
  // zero, and straight-line issue keeps the compiler's load counting exact (a load under a
  // branch makes it wait for everything at the join)
  const __amdgpu_buffer_rsrc_t bres = make_rsrc(j.Bpk, (uint64_t)bp_total * 2);
  auto fetch_b = [&](int c) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int64_t idx = (int64_t)c * CH + (int64_t)(i * kHiloWaves * 64 + threadIdx.x) * 8;
      bst[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(bres, (int)(idx * 2), 0, 0));
    }
  };
  auto stash_b = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      *reinterpret_cast<u32x4*>(bs + buf * CH + (i * kHiloWaves * 64 + threadIdx.x) * 8) = bst[i];
  };

  // X chunk xc of this wave's rows. A piece at or past column p (and a chunk past the last)
  // would read the row's padding or the next rows' bytes, real traffic that is thrown away:
  // its offset is put past every resource's end, so it reads zero and moves nothing.
  struct XRegs { u32x4 v[4][PL]; };
  auto load_x = [&](int xc, XRegs& x) {
    const bool live = 64 * xc + 8 * piece < p;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t off = live ? xoff[i] + 128 * (uint32_t)xc : 0xFFFFFFF0u;
      x.v[i][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rh, (int)off, 0, AUX));
      if (LO) x.v[i][PL - 1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rl, (int)off, 0, AUX));
    }
  };
  // zero the elements of this lane's 8 columns 64 xc + 8 piece .. that lie past p
  auto mask_tail = [&](int xc, XRegs& x) {
    const int lim = p - (64 * xc + 8 * piece);
    u32x4 mk;
#pragma unroll
    for (int d = 0; d < 4; ++d)
      mk[d] = (2 * d < lim ? 0x0000FFFFu : 0u) | (2 * d + 1 < lim ? 0xFFFF0000u : 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int pl = 0; pl < PL; ++pl) x.v[i][pl] &= mk;
  };
  u16* xw = bs + 2 * CH + w * PL * 2048;          // this wave's 32 rows x 64 columns of each plane
  const int xput = (lane >> 3) * 64;              // row lane / 8 of instruction 0
  auto stash_x = [&](const XRegs& x) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int pos = piece ^ ((4 * i + (lane >> 4)) & 7);
#pragma unroll
      for (int pl = 0; pl < PL; ++pl)
        *reinterpret_cast<u32x4*>(xw + pl * 2048 + xput + i * 512 + 8 * pos) = x.v[i][pl];
    }
  };
  // k step 2 xc + h of the staged chunk with fragment kk of the B buffer
  auto step = [&](int h, const u16* bk) {
    bf16x8 bh[NB], bl[NB], ah[MB], al[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const u16* f = xw + (16 * mb + m) * 64 + 8 * ((4 * h + g) ^ ((m >> 1) & 7));
      ah[mb] = as_frag(*reinterpret_cast<const u32x4*>(f));
      if (LO) al[mb] = as_frag(*reinterpret_cast<const u32x4*>(f + 2048));
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      bh[nb] = as_frag(*reinterpret_cast<const u32x4*>(bk + nb * 1024));
      bl[nb] = as_frag(*reinterpret_cast<const u32x4*>(bk + nb * 1024 + 512));
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mma(ah[mb], bh[nb], acc[mb][nb]);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mma(ah[mb], bl[nb], acc[mb][nb]);
    if (LO) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mma(al[mb], bh[nb], acc[mb][nb]);
    }
  };
  // Register set q holds chunks q, q + kXDepth, ...; it is reloaded right after its chunk is
  // stored to LDS, so kXDepth - 1 chunks of loads stay in flight per wave and one more is
  // issued while a chunk is used. The index is static in the unrolled loop, so no register is
  // copied (a copy of a register a load has not yet filled would wait for that load).
  constexpr int XB = BST / 2;                     // X chunks per B chunk
  constexpr int UN = XD > XB ? XD / XB : 1;       // B chunks per turn of the register ring
  XRegs x[XD];
  fetch_b(0);
  stash_b(0);
#pragma unroll
  for (int q = 0; q < XD; ++q) load_x(q, x[q]);
  __syncthreads();
  for (int c0 = 0; c0 < nch; c0 += UN) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int c = c0 + u;
      if (c >= nch) break;
      fetch_b(c + 1);
      const u16* bc = bs + (c & 1) * CH + lane * 8;
#pragma unroll
      for (int b = 0; b < XB; ++b) {
        const int xc = c * XB + b;
        XRegs& xr = x[(u * XB + b) % XD];
        if (xc == nxc - 1 && (p & 7)) mask_tail(xc, xr);
        __builtin_amdgcn_wave_barrier();          // the previous chunk's operands are read
        stash_x(xr);
        load_x(xc + XD, xr);
        __builtin_amdgcn_wave_barrier();
        if (2 * xc < nks) step(0, bc + (2 * b) * NB * 1024);
        if (2 * xc + 1 < nks) step(1, bc + (2 * b + 1) * NB * 1024);
      }
      stash_b((c + 1) & 1);
      __syncthreads();
    }
  }

  softmax_residuals<NB, GROUP>(j, rb, acc, ylab, lacc);
}

// The logits of a problem of few rows, which are one workgroup's: the latency of its chain of k steps
// bounds them, not the reading of X. The A operand comes straight from global memory, kFewSteps - 1 k
// steps ahead of the MFMAs: lane l loads the 8 consecutive columns 32 s + 8 (l / 16) .. of row l % 16
// of each M block, the A input layout, without the turn through LDS that whole lines take in
// logits_rows. B as there; same order of sums. A gradient with hi + lo planes, here and there: n = 12,
// p = 5620, K = 33 83 and 117 us; n = 31, p = 11617, K = 20 101 and 147. With more rows the lines
// gain on it (p of 1500 to 14000, K = 8, n = 80: 0.98 of the time and 0.90, n = 88: 0.98 and 0.85; K = 50,
// whose B chunks are half as long there, n = 88: 0.93 and 1.16, n = 128: 0.96 and 1.01).
constexpr int kFewSteps = 4;
template <int NB> constexpr int few_lds_elems() { return 2 * kFewSteps * NB * 1024; }
template <int NB, int GROUP, bool LO>
__device__ __forceinline__ void logits_few_rows(const Job& j, double (&lacc)[NB / GROUP], u16* __restrict__ bs) {
  constexpr int CH = kFewSteps * NB * 1024;         // u16 per chunk (hi and lo fragments)
  constexpr int PER = CH / 8 / (kHiloWaves * 64);   // 16-byte pieces per thread per chunk
  static_assert(CH / 8 % (kHiloWaves * 64) == 0, "a B chunk is a whole number of 16-byte pieces per thread");
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int64_t n = j.n;
  const int p = j.p;
  const int nks = (p + 31) / 32;
  constexpr int MB = kHiloMB;
  f32x4 acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // X fragments come from branch-free buffer loads whose resource ends at row n, so rows past
  // n read as zero; columns past p are zeroed in registers on the last (ragged) k step.
  const uint64_t rem = (uint64_t)n * j.ldx * 2;
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(j.Xhi, rem);
  const __amdgpu_buffer_rsrc_t rl = make_rsrc(LO ? j.Xlo : j.Xhi, LO ? rem : 0);
  uint32_t xoff[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
    xoff[mb] = (uint32_t)(((int64_t)(w * 16 * MB + 16 * mb + m) * j.ldx + 8 * g) * 2);
  // labels of this lane's rows, loaded now so their latency hides behind the k loop
  // (rows past n read as zero and are not used)
  const __amdgpu_buffer_rsrc_t yres = make_rsrc(j.y, (uint64_t)n * 4);
  int ylab[MB][4];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      ylab[mb][i] = __builtin_amdgcn_raw_buffer_load_b32(
          yres, (int)((w * 16 * MB + 16 * mb + 4 * g + i) * 4), 0, 0);
  const int nch = (nks + kFewSteps - 1) / kFewSteps;
  const int64_t bp_total = (int64_t)nks * NB * 1024;
  u32x4 bst[PER];
  // every load below is issued unconditionally: buffer loads past a resource's end read
  // zero, and straight-line issue keeps the compiler's load counting exact (a load under a
  // branch makes it wait for everything at the join)
  const __amdgpu_buffer_rsrc_t bres = make_rsrc(j.Bpk, (uint64_t)bp_total * 2);
  auto fetch_b = [&](int c) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int64_t idx = (int64_t)c * CH + (int64_t)(i * kHiloWaves * 64 + threadIdx.x) * 8;
      bst[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(bres, (int)(idx * 2), 0, 0));
    }
  };
  auto stash_b = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      *reinterpret_cast<u32x4*>(bs + buf * CH + (i * kHiloWaves * 64 + threadIdx.x) * 8) = bst[i];
  };

  // A fragments of k step ks. A step at or past nks (the ring's refills during the last
  // chunk) would read the next rows' bytes, real traffic that is thrown away: those loads
  // take an empty resource instead (still issued, so the issue stays branch-free).
  const __amdgpu_buffer_rsrc_t rz = make_rsrc(j.Xhi, 0);
  auto load_a = [&](int ks, u32x4 (&ah)[MB], u32x4 (&al)[MB]) {
    const bool live = ks < nks;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      ah[mb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(live ? rh : rz, (int)(xoff[mb] + 64 * ks), 0, 0));
      if (LO) al[mb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(live ? rl : rz, (int)(xoff[mb] + 64 * ks), 0, 0));
    }
  };
  // zero the elements of this lane's 8 columns 32 ks + 8 g .. that lie past p
  auto mask_tail = [&](int ks, u32x4 (&ah)[MB], u32x4 (&al)[MB]) {
    const int lim = p - (32 * ks + 8 * g);
    u32x4 mk;
#pragma unroll
    for (int d = 0; d < 4; ++d)
      mk[d] = (2 * d < lim ? 0x0000FFFFu : 0u) | (2 * d + 1 < lim ? 0xFFFF0000u : 0u);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      ah[mb] &= mk;
      if (LO) al[mb] &= mk;
    }
  };
  // X fragments kFewSteps k steps ahead in a ring of kFewSteps register sets: set kk holds
  // step ks = c kFewSteps + kk of chunk c and is reloaded with step ks + kFewSteps right after
  // its MFMAs, so kFewSteps - 1 steps of loads stay in flight per wave while one is used.
  // The ring index is static in the unrolled chunk, so no register is copied (a copy of a
  // register a load has not yet filled would wait for that load).
  u32x4 xh[kFewSteps][MB], xl[kFewSteps][MB];
  fetch_b(0);
  stash_b(0);
#pragma unroll
  for (int kk = 0; kk < kFewSteps; ++kk) load_a(kk, xh[kk], xl[kk]);
  __syncthreads();
  for (int c = 0; c < nch; ++c) {
    fetch_b(c + 1);
    const u16* bc = bs + (c & 1) * CH + lane * 8;
#pragma unroll
    for (int kk = 0; kk < kFewSteps; ++kk) {
      const int ks = c * kFewSteps + kk;
      if (ks == nks - 1 && (p & 31)) mask_tail(ks, xh[kk], xl[kk]);
      bf16x8 bh[NB], bl[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const u16* f = bc + (kk * NB + nb) * 1024;
        bh[nb] = as_frag(*reinterpret_cast<const u32x4*>(f));
        bl[nb] = as_frag(*reinterpret_cast<const u32x4*>(f + 512));
      }
      if (ks < nks) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            acc[mb][nb] = mma(as_frag(xh[kk][mb]), bh[nb], acc[mb][nb]);
            acc[mb][nb] = mma(as_frag(xh[kk][mb]), bl[nb], acc[mb][nb]);
            if (LO) acc[mb][nb] = mma(as_frag(xl[kk][mb]), bh[nb], acc[mb][nb]);
          }
      }
      load_a(ks + kFewSteps, xh[kk], xl[kk]);
    }
    stash_b((c + 1) & 1);
    __syncthreads();
  }

  softmax_residuals<NB, GROUP>(j, 0, acc, ylab, lacc);
}

// Gradient partial X^T R of the 32 NW columns from c0 over rows [rbeg, rend) (rbeg a
// multiple of 32), written to gp: element (column j, class kk of group q) at
// gp[q cstride + j K + kk].
//
// Loads bound it: every column block of a slice reads the slice's packed residuals again (from
// the L2), 256 bytes per row and 4 class blocks beside 1 KB of X for 256 columns. With 128
// columns per workgroup those reads took 60-85 us of the kernel's time (timed without them):
// n = 200000, p = 4096, K = 64 took 626 us there and 532 here (6.2 TB/s), a batch of 16
// problems x 4 chains 360 and 325.
//
// Stages of 32 rows (both X planes, 32 x 256 bf16 each, and the matching packed residual
// fragments) are loaded into registers two stages ahead of the math and stored to one of
// two LDS buffers one stage ahead, so two stages of loads stay in flight per workgroup.
// Wave w owns columns 32 w .. 32 w + 31 (two 16-column M blocks); the MFMA A input wants,
// per lane, 8 consecutive ROWS of one column: two transposing LDS reads (ds_read_b64_tr_b16,
// each turning 4 rows x 16 columns of a 16-lane group) per operand, in place of eight 16-bit
// reads and their packing, which with the residual reads had filled the LDS pipe for most of
// the time that streaming a stage takes. The 16-byte chunks of a staged row are XOR-swizzled
// by 2 (row % 4 + 4 ((row / 8) % 2)), so that the eight rows a read touches at once fall in
// different banks. Rows outside the slice and columns past p load as zero.
constexpr int grad_plane(int nw) { return 32 * grad_cols(nw); }   // u16 of one plane per stage
template <int NB, bool LO, int NW> constexpr int grad_stage_elems() { return (LO ? 2 : 1) * grad_plane(NW) + NB * 1024; }
// residual u16 per thread and piece: the stage's NB * 1024 over the threads, 16 bytes at most
template <int N_> struct RPieceOf;
template <> struct RPieceOf<2> { typedef uint32_t type; static constexpr int N = 2; };
template <> struct RPieceOf<4> { typedef uint2 type; static constexpr int N = 4; };
template <> struct RPieceOf<8> { typedef u32x4 type; static constexpr int N = 8; };
template <int NB, int NW> struct RPiece : RPieceOf<(NB * 16 / NW < 8 ? NB * 16 / NW : 8)> {};

template <int NB, int GROUP, bool LO, int AUX, int NW>
__device__ __forceinline__ void grad_block(const Job& j, int64_t c0, int64_t rbeg, int64_t rend,
                                          float* __restrict__ gp, int64_t cstride,
                                          u16* __restrict__ xs) {
  constexpr int PL = LO ? 2 : 1, GC = grad_cols(NW), TH = 64 * NW, GP = grad_plane(NW);
  constexpr int XST = PL * GP;                  // u16 of X per stage
  constexpr int ST = grad_stage_elems<NB, LO, NW>();
  constexpr int RN = RPiece<NB, NW>::N;               // residual u16 per thread per piece
  constexpr int RP = NB * 1024 / (TH * RN);      // residual pieces per thread per stage
  typedef typename RPiece<NB, NW>::type rtype;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int m = lane & 15, g = lane >> 4;
  const int p = j.p, K = j.K;
  const int64_t nst = rend > rbeg ? (rend - rbeg + 31) / 32 : 0;

  // staging: thread t moves 16-byte chunk sc of rows sr and sr + 16 of each plane, and
  // residual pieces t, t + TH, ...
  const int sr = threadIdx.x / (GC / 8), sc = threadIdx.x % (GC / 8);
  const int64_t col = c0 + 8 * sc;
  struct Regs { u32x4 x[2][PL]; rtype r[RP]; };
  // Branch-free buffer loads: the X resource of a stage starts at its first row and ends
  // at the slice's last row (rows outside the slice read as zero; columns past p only feed
  // gradient columns that are not written); the residual resource covers the packed
  // buffer, so stages past the end read zero.
  const uint64_t rpk_bytes = (uint64_t)((j.n + kHiloRows - 1) / kHiloRows) * (kHiloRows / 32) * NB * 2048;
  const __amdgpu_buffer_rsrc_t rres = make_rsrc(j.Rpk, rpk_bytes);
  // a chunk at or past column p (the last column block of a problem whose p is not a
  // multiple of 32 NW) would fetch the row's padding or the next row's bytes for columns that
  // are never written: its offset is put out of the resource's range, so it reads zero and
  // moves nothing
  uint32_t xo[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
    xo[h] = col < p ? (uint32_t)(((int64_t)(sr + 16 * h) * j.ldx + col) * 2) : 0xFFFFFFF0u;
  auto fetch = [&](int64_t k, Regs& R) {
    const int64_t row0 = rbeg + 32 * k;
    const bool real = k < nst;
    const uint64_t xbytes = real ? (uint64_t)(rend - row0) * j.ldx * 2 : 0;
    const int64_t xbase = real ? row0 * j.ldx : 0;
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) {
      const __amdgpu_buffer_rsrc_t xr = make_rsrc((pl ? j.Xlo : j.Xhi) + xbase, xbytes);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        R.x[h][pl] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)xo[h], 0, AUX));
    }
    const uint32_t roff = (uint32_t)((real ? row0 / 32 : (int64_t)(rpk_bytes / (NB * 2048))) * NB * 2048);
#pragma unroll
    for (int i = 0; i < RP; ++i) {
      const int off = (int)(roff + (i * TH + threadIdx.x) * RN * 2);
      if constexpr (RN == 2)
        R.r[i] = (rtype)__builtin_amdgcn_raw_buffer_load_b32(rres, off, 0, 0);
      else if constexpr (RN == 8)
        R.r[i] = __builtin_bit_cast(rtype, __builtin_amdgcn_raw_buffer_load_b128(rres, off, 0, 0));
      else
        R.r[i] = __builtin_bit_cast(rtype, __builtin_amdgcn_raw_buffer_load_b64(rres, off, 0, 0));
    }
  };
  // XOR of a row's 16-byte chunk index (the same for rows q and q + 4); two 64-column rows share
  // the 256 bytes that a pair of chunks is spread over
  auto swizzle = [](int q) {
    return NW == 2 ? 2 * (((q >> 1) & 1) | ((q >> 2) & 2)) : 2 * ((q & 3) | ((q >> 1) & 4));
  };
  auto stash = [&](const Regs& R, u16* buf) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int q = sr + 16 * h;
      const int pos = sc ^ swizzle(q);
#pragma unroll
      for (int pl = 0; pl < PL; ++pl)
        *reinterpret_cast<u32x4*>(buf + pl * GP + q * GC + 8 * pos) = R.x[h][pl];
    }
#pragma unroll
    for (int i = 0; i < RP; ++i)
      *reinterpret_cast<rtype*>(buf + XST + (i * TH + threadIdx.x) * RN) = R.r[i];
  };

  f32x4 acc[2][NB];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // transposing reads: lane 16 g + m supplies row 8 g + m / 4 (+ 4), columns 4 (m % 4) .. + 3 of
  // the M block, and receives column m of rows 8 g .. 8 g + 3 (+ 4)
  const int trow = 8 * g + (m >> 2);
  int tcol[2];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
    tcol[mb] = 8 * ((4 * w + 2 * mb + ((m >> 1) & 1)) ^ swizzle(trow)) + 4 * (m & 1);
  auto compute = [&](const u16* cur) {
    bf16x8 bh[NB], bl[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      bh[nb] = as_frag(*reinterpret_cast<const u32x4*>(cur + XST + nb * 1024 + lane * 8));
      bl[nb] = as_frag(*reinterpret_cast<const u32x4*>(cur + XST + nb * 1024 + 512 + lane * 8));
    }
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      bf16x8 af[PL];
#pragma unroll
      for (int pl = 0; pl < PL; ++pl) {
        const u16* t = cur + pl * GP + trow * GC + tcol[mb];
        af[pl] = as_frag(tr_pair(t, t + 4 * GC));
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        acc[mb][nb] = mma(af[0], bh[nb], acc[mb][nb]);
        acc[mb][nb] = mma(af[0], bl[nb], acc[mb][nb]);
        if (LO) acc[mb][nb] = mma(af[PL - 1], bh[nb], acc[mb][nb]);
      }
    }
  };

  // register sets: stage k in ra (k even) or rb (k odd), loaded two steps before its use
  Regs ra, rb;
  fetch(0, ra);
  fetch(1, rb);
  // in pairs, the second of an odd count a stage of zeros (a branch in the middle cost a second
  // set of accumulator registers)
  for (int64_t k = 0; k < nst; k += 2) {
    stash(ra, xs);
    __syncthreads();
    fetch(k + 2, ra);
    compute(xs);
    stash(rb, xs + ST);
    __syncthreads();
    fetch(k + 3, rb);
    compute(xs + ST);
  }
  __syncthreads();   // the buffers are reused by the caller's next item

  // lane l holds G[column 4 (l / 16) + i of the M block][class 16 nb + l % 16]
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t jc = c0 + 32 * w + 16 * mb + 4 * g + i;
      if (jc >= p) continue;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int kk = 16 * (nb % GROUP) + m;
        if (kk < K) gp[(nb / GROUP) * cstride + jc * K + kk] = acc[mb][nb][i];
      }
    }
}

// XCD-aware item order of the gradient kernels. Workgroup w of a launch runs on XCD w % 8,
// and consecutive items (the column blocks of one row slice) read the same packed residual
// rows, so they should share an XCD's L2: position `it` of the launch order is mapped to
// item (it % 8 + 8 (it / 8 / G)) G + (it / 8) % G, which gives XCD x the chunks x, x + 8, ...
// of G consecutive items. It is a bijection of [0, round_up(total, 8 G)); positions whose
// item is >= total do nothing.
__device__ __forceinline__ int64_t xcd_item(int64_t it, int G) {
  const int64_t x = it % kXcds, l = it / kXcds;
  return (x + kXcds * (l / G)) * G + l % G;
}

__device__ __forceinline__ Job job_of(const HiloArgs& a) {
  return Job{a.Xhi, a.Xlo, a.ldx, a.y, a.n, a.p, a.K, static_cast<const float*>(a.B), a.Bpk, a.Rpk, a.pin};
}

// ---------------------------------------------------------------------------------------
// Single-problem kernels (one softmax group spanning all NB class blocks).
template <int NB>
__global__ __launch_bounds__(256) void pack_b_kernel(HiloArgs a) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)((a.p + 31) / 32) * NB * 64) return;
  pack_b_body<NB, NB>(job_of(a), t);
}

template <int NB, bool LO>
__global__ __launch_bounds__(kHiloWaves * 64) void hilo_logits(HiloArgs a) {
  constexpr int ROWS = kHiloRows;
  __shared__ double lsum[kHiloWaves];
  __shared__ __attribute__((aligned(16))) u16 bs[logits_lds_elems<NB, LO>()];
  const Job j = job_of(a);
  const int64_t nrb = (a.n + ROWS - 1) / ROWS;
  double lacc[1] = {0.0};
  for (int64_t rb = blockIdx.x; rb < nrb; rb += gridDim.x) {
    if (hot_slice(rb * ROWS / a.rows_per_split, a.hot)) logits_rows<NB, NB, LO, kKeep>(j, rb, lacc, bs);
    else logits_rows<NB, NB, LO, kStream>(j, rb, lacc, bs);
  }
  const double v = wave_sum(lacc[0]);
  if ((threadIdx.x & 63) == 0) lsum[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < kHiloWaves; ++i) t += lsum[i];
    a.lpart[blockIdx.x] = t;
  }
}

template <int NB, bool LO>
__global__ __launch_bounds__(kHiloWaves * 64) void hilo_logits_few(HiloArgs a) {
  __shared__ double lsum[kHiloWaves];
  __shared__ __attribute__((aligned(16))) u16 bs[few_lds_elems<NB>()];
  double lacc[1] = {0.0};
  logits_few_rows<NB, NB, LO>(job_of(a), lacc, bs);
  const double v = wave_sum(lacc[0]);
  if ((threadIdx.x & 63) == 0) lsum[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < kHiloWaves; ++i) t += lsum[i];
    a.lpart[0] = t;
  }
}

// One workgroup of NW waves per (32 NW-column block, row slice) item, items slice-major (the
// column blocks of a slice consecutive) in the XCD-aware order; the launch has xcd_span(items,
// gcols) workgroups.
template <int NB, bool LO, int NW>
__global__ __launch_bounds__(64 * NW, 2) void hilo_grad(HiloArgs a, int gcols) {
  __shared__ __attribute__((aligned(16))) u16 xs[2 * grad_stage_elems<NB, LO, NW>()];
  const int64_t it = xcd_item(blockIdx.x, gcols);
  if (it >= (int64_t)gcols * a.nsplit) return;
  const int64_t cb = it % gcols, sl = it / gcols;
  const int64_t rbeg = sl * a.rows_per_split;
  const int64_t rend = rbeg + a.rows_per_split < a.n ? rbeg + a.rows_per_split : a.n;
  if (hot_slice(sl, a.hot)) grad_block<NB, NB, LO, kKeep, NW>(job_of(a), cb * grad_cols(NW), rbeg, rend, a.gpart + sl * a.gstride, 0, xs);
  else grad_block<NB, NB, LO, kStream, NW>(job_of(a), cb * grad_cols(NW), rbeg, rend, a.gpart + sl * a.gstride, 0, xs);
}

// ---------------------------------------------------------------------------------------
// Batched kernels: every problem of a batch, NB chains each (one class block per chain),
// in one persistent launch per phase. Work items are numbered table entry by table entry
// (the host orders the entries by decreasing p); item i belongs to entry b with
// first[b] <= i < first[b + 1].
__device__ __forceinline__ int find_problem(const int32_t* first, int nprob, int64_t item) {
  int lo = 0, hi = nprob;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (first[mid] <= item) lo = mid; else hi = mid;
  }
  return lo;
}

// A value that is the same in every lane, moved to scalar registers: the table's entries are
// loaded by vector loads (the kernels' own stores could alias them), and would hold, with all
// that is computed from them, vector registers for the whole item.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 | lo);
}
template <typename T> __device__ __forceinline__ T* uniform(T* p) {
  return reinterpret_cast<T*>(uniform((int64_t)reinterpret_cast<uintptr_t>(p)));
}

__device__ __forceinline__ Job job_of(const BatchProb& b, const float* B) {
  return Job{uniform(b.Xhi), uniform(b.Xlo), uniform(b.ldx), uniform(b.y), uniform(b.n), uniform(b.p), uniform(b.K),
             B, uniform(b.Bpk), uniform(b.Rpk), uniform(b.pin)};
}

template <int NB, int GROUP>
__global__ __launch_bounds__(256) void batch_pack(BatchArgs a) {
  const int64_t total = a.first_pack[a.nprob];
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
    const int b = find_problem(a.first_pack, a.nprob, t);
    const BatchProb& P = a.probs[b];
    pack_b_body<NB, GROUP>(job_of(P, a.at_current ? P.B : P.Bp), t - a.first_pack[b]);
  }
}

// FEW: every problem has few_rows rows at most (one item each).
template <int NB, int GROUP, bool LO, bool FEW>
__global__ __launch_bounds__(kHiloWaves * 64, 2) void batch_logits(BatchArgs a) {
  constexpr int NC = NB / GROUP;                  // chains
  __shared__ double lsum[kHiloWaves][NC];
  __shared__ __attribute__((aligned(16))) u16 bs[FEW ? few_lds_elems<NB>() : logits_lds_elems<NB, LO>()];
  const int64_t total = a.first_logits[a.nprob];
  for (int64_t it = blockIdx.x; it < total; it += gridDim.x) {
    const int b = find_problem(a.first_logits, a.nprob, it);
    const BatchProb& P = a.probs[uniform(b)];
    const int64_t rb = uniform(it - a.first_logits[b]);
    double lacc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) lacc[c] = 0.0;
    const Job j = job_of(P, nullptr);
    if constexpr (FEW) logits_few_rows<NB, GROUP, LO>(j, lacc, bs);
    else if (hot_slice(uniform(P.slice0) + rb * kHiloRows / uniform(P.rps), uniform(P.hot))) logits_rows<NB, GROUP, LO, kKeep>(j, rb, lacc, bs);
    else logits_rows<NB, GROUP, LO, kStream>(j, rb, lacc, bs);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double v = wave_sum(lacc[c]);
      if ((threadIdx.x & 63) == 0) lsum[threadIdx.x >> 6][c] = v;
    }
    __syncthreads();
    if (threadIdx.x < NC) {
      double t = 0.0;
      for (int i = 0; i < kHiloWaves; ++i) t += lsum[i][threadIdx.x];
      P.lpart[rb * NC + threadIdx.x] = t;
    }
    __syncthreads();
  }
}

template <int NB, int GROUP, bool LO, int NW>
__global__ __launch_bounds__(64 * NW, 2) void batch_grad(BatchArgs a) {
  __shared__ __attribute__((aligned(16))) u16 xs[2 * grad_stage_elems<NB, LO, NW>()];
  const int64_t total = a.first_grad[a.nprob];
  const int64_t span = xcd_span(total, grad_chunk(NW));
  for (int64_t pos = blockIdx.x; pos < span; pos += gridDim.x) {
    const int64_t it = xcd_item(pos, grad_chunk(NW));
    if (it >= total) continue;
    const int b = find_problem(a.first_grad, a.nprob, it);
    const BatchProb& P = a.probs[uniform(b)];
    const int64_t k = uniform(it - a.first_grad[b]), gcols = uniform(P.gcols), rps = uniform(P.rps);
    const int64_t cb = k % gcols, s = k / gcols;
    const Job j = job_of(P, nullptr);
    const int64_t rbeg = s * rps, rend = rbeg + rps < j.n ? rbeg + rps : j.n;
    float* gp = uniform(P.gpart + s * P.gstride);
    if (hot_slice(uniform(P.slice0) + s, uniform(P.hot))) grad_block<NB, GROUP, LO, kKeep, NW>(j, cb * grad_cols(NW), rbeg, rend, gp, uniform(P.cstride), xs);
    else grad_block<NB, GROUP, LO, kStream, NW>(j, cb * grad_cols(NW), rbeg, rend, gp, uniform(P.cstride), xs);
  }
}

}  // namespace

template <typename Tin>
hipError_t launch_split(const Tin* X, int64_t ldx, int64_t n, int64_t p, uint16_t* hi,
                        uint16_t* lo, int64_t ldo, hipStream_t s) {
  // groups per workgroup; grids beyond 2^31 workgroups take more rows each
  const int64_t gpr = ldo / 8, all = n * gpr;
  const int64_t fit = p < 8 ? 256 : std::max<int64_t>(256, all / kSplitWorkgroups / 256 * 256);
  const int64_t want = std::min<int64_t>(kSplitGroups, fit);
  const int64_t span = want < kSplitGroups && gpr > want ? std::max(want, (gpr + 0x7FFF) / 0x8000) : std::min(gpr, kSplitSpan);
  const int64_t rows = std::max<int64_t>({1, want / gpr, (n + 0x3FFFFFFF) / 0x40000000});
  const dim3 grid((unsigned)((n + rows - 1) / rows), (unsigned)((gpr + span - 1) / span));
  if (want == 256)
    hipLaunchKernelGGL((split_kernel<Tin, 1>), grid, dim3(256), 0, s, X, ldx, n, p, hi, lo, ldo, (uint32_t)rows, span);
  else
    hipLaunchKernelGGL((split_kernel<Tin, kSplitUnroll>), grid, dim3(256), 0, s, X, ldx, n, p, hi, lo, ldo, (uint32_t)rows, span);
  return hipGetLastError();
}
template hipError_t launch_split<float>(const float*, int64_t, int64_t, int64_t, uint16_t*, uint16_t*, int64_t, hipStream_t);
template hipError_t launch_split<double>(const double*, int64_t, int64_t, int64_t, uint16_t*, uint16_t*, int64_t, hipStream_t);

template <int NB, int GROUP, bool LO>
static hipError_t launch_batch_t(const BatchArgs& a, bool few, int grad_waves, const int grid[3], bool pack, hipStream_t s) {
  if (pack) hipLaunchKernelGGL((batch_pack<NB, GROUP>), dim3(grid[0]), dim3(256), 0, s, a);
  if (few) hipLaunchKernelGGL((batch_logits<NB, GROUP, LO, true>), dim3(grid[1]), dim3(kHiloWaves * 64), 0, s, a);
  else hipLaunchKernelGGL((batch_logits<NB, GROUP, LO, false>), dim3(grid[1]), dim3(kHiloWaves * 64), 0, s, a);
  switch (grad_waves) {
    case 8: hipLaunchKernelGGL((batch_grad<NB, GROUP, LO, 8>), dim3(grid[2]), dim3(512), 0, s, a); break;
    case 4: hipLaunchKernelGGL((batch_grad<NB, GROUP, LO, 4>), dim3(grid[2]), dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((batch_grad<NB, GROUP, LO, 2>), dim3(grid[2]), dim3(128), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// chains x group class blocks (group = 16-class blocks per chain), at most 4 in all
hipError_t launch_batch_pass(const BatchArgs& a, int chains, int group, bool lo, bool few, int grad_waves, const int grid[3], bool pack, hipStream_t s) {
#define HMC_BATCH(C_, G_)                                                                 \
  if (chains == C_ && group == G_)                                                        \
    return lo ? launch_batch_t<C_ * G_, G_, true>(a, few, grad_waves, grid, pack, s)                      \
              : launch_batch_t<C_ * G_, G_, false>(a, few, grad_waves, grid, pack, s);
  HMC_BATCH(1, 1) HMC_BATCH(2, 1) HMC_BATCH(4, 1) HMC_BATCH(1, 2) HMC_BATCH(2, 2) HMC_BATCH(1, 4)
#undef HMC_BATCH
  return hipErrorInvalidValue;
}

template <int NB, bool LO>
static hipError_t launch_hilo_t(const HiloArgs& a, int logits_wg, int grad_waves, bool pack, hipStream_t s) {
  const int gcols = (a.p + grad_cols(grad_waves) - 1) / grad_cols(grad_waves);
  const int nks = (a.p + 31) / 32;
  const int packs = (nks * NB * 64 + 255) / 256;
  if (pack) hipLaunchKernelGGL(pack_b_kernel<NB>, dim3(packs), dim3(256), 0, s, a);
  if (a.n <= few_rows(NB)) hipLaunchKernelGGL((hilo_logits_few<NB, LO>), dim3(1), dim3(kHiloWaves * 64), 0, s, a);
  else hipLaunchKernelGGL((hilo_logits<NB, LO>), dim3(logits_wg), dim3(kHiloWaves * 64), 0, s, a);
  const int64_t span = xcd_span((int64_t)gcols * a.nsplit, gcols);
  if (grad_waves == 2) hipLaunchKernelGGL((hilo_grad<NB, LO, 2>), dim3((unsigned)span), dim3(128), 0, s, a, gcols);
  else if (grad_waves == 4) hipLaunchKernelGGL((hilo_grad<NB, LO, 4>), dim3((unsigned)span), dim3(256), 0, s, a, gcols);
  else hipLaunchKernelGGL((hilo_grad<NB, LO, 8>), dim3((unsigned)span), dim3(512), 0, s, a, gcols);
  return hipGetLastError();
}

hipError_t launch_hilo(const HiloArgs& a, int nb, bool lo, int logits_wg, int grad_waves, bool pack, hipStream_t s) {
  switch (nb * 2 + (lo ? 1 : 0)) {
    case 2: return launch_hilo_t<1, false>(a, logits_wg, grad_waves, pack, s);
    case 3: return launch_hilo_t<1, true>(a, logits_wg, grad_waves, pack, s);
    case 4: return launch_hilo_t<2, false>(a, logits_wg, grad_waves, pack, s);
    case 5: return launch_hilo_t<2, true>(a, logits_wg, grad_waves, pack, s);
    case 8: return launch_hilo_t<4, false>(a, logits_wg, grad_waves, pack, s);
    case 9: return launch_hilo_t<4, true>(a, logits_wg, grad_waves, pack, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace hmcx
