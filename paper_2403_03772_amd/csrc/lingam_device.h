// Device helpers shared by the gfx950 kernel sources of the library (not
// installed; each source gets its own copies in an unnamed namespace).
#pragma once

#include "lingam_internal.h"

#include <math.h>

namespace lg {
namespace {

// Constants of the maximum-entropy approximation of differential entropy.
constexpr double kK1 = 79.047;
constexpr double kK2 = 7.4129;
constexpr double kGamma = 0.37457;
constexpr double kHnu = 1.41893853320467274178;  // (1 + ln(2 pi)) / 2
constexpr double kLn2 = 0.69314718055994530942;
constexpr double kLog2e = 1.44269504088896340736;
constexpr double kCollinear = 1e-12;  // |rho| >= 1 - kCollinear is degenerate
constexpr int kLogBlock = 32;         // samples per lane folded into one log2 (product <= 2^32)
constexpr int kSumBlock = 16;         // ... in the pair kernels' separate form
constexpr float kS1Start = 9.0f;      // start value (negated) of each lane's log cosh sum

// beside a variable's five moments: the largest |z|, and the sum of its FP32 copy
constexpr int kMomTop = 5;
constexpr int kMomSum = 6;

constexpr int32_t kStInvalid = -1;
constexpr int32_t kStDegenerate = -2;

template <typename T>
__host__ __device__ inline T* at(char* ws, size_t off) {
  return reinterpret_cast<T*>(ws + off);
}

__device__ inline void set_status(Ctrl* c, int32_t s) { atomicCAS(&c->status, 0, s); }

// The order or row map of a call was refused by its check (nothing may be read or
// written through it); ctrl NULL: not checked.
__device__ inline bool refused(const Ctrl* ctrl) { return ctrl && ctrl->status == kStInvalid; }

// Job blockIdx.z's copy of a region, the jobs' workspaces `bytes` apart.
template <class T>
__device__ inline T* job_at(T* p, size_t bytes) {
  return (T*)((char*)p + blockIdx.z * bytes);
}

__device__ inline double entropy_from_moments(double e_lc, double e_g) {
  const double a = e_lc - kGamma;
  return kHnu - kK1 * a * a - kK2 * e_g * e_g;
}

// One evaluation (one residual direction at one sample).  See the header.
__device__ __forceinline__ void eval_dir(float x, float y, float r, float c1h, float c1l,
                                         float& P, float& S1, float& S2) {
  const float kM2 = (float)(-1.0 / (8.0 * kLog2e));  // rounds with relative error 2.7e-9
  const float t = fmaf(-r, y, x);
  const float at = fabsf(t);
  const float m1 = fmaf(c1h, at, c1l * at);
  const float e1 = __builtin_amdgcn_exp2f(m1);
  P = fmaf(P, e1, P);
  S1 = fmaf(m1, -0.5f, S1);
  const float m2 = (kM2 * m1) * m1;
  const float e2 = __builtin_amdgcn_exp2f(m2);
  S2 = fmaf(t, e2, S2);
}

// The two FP32 values around c (equal when c is a float) and how many of the
// 64 lanes take the upper one so that the lanes' mean is c to 1/128 of a
// float spacing.
__device__ inline void dither_float(double c, float& lo, float& hi, int& n_hi) {
  const float f = (float)c;
  if ((double)f == c) {
    lo = hi = f;
    n_hi = 0;
    return;
  }
  const float g = (double)f < c ? nextafterf(f, INFINITY) : nextafterf(f, -INFINITY);
  lo = fminf(f, g);
  hi = fmaxf(f, g);
  // hi - lo is a power of two: scale by its exponent instead of dividing
  const double gap = (double)hi - (double)lo;
  n_hi = (int)rint(ldexp(c - (double)lo, 6 - ilogb(gap)));
}

// 2^(j / 64), rounded to FP64.
constexpr int kExpTable = 64;
__device__ constexpr double kExp2[kExpTable] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0};

// The table in LDS (as many threads as it has entries at least); the caller's next
// barrier orders it.
__device__ inline void stage_exp(double (&tab)[kExpTable]) {
  if (threadIdx.x < kExpTable) tab[threadIdx.x] = kExp2[threadIdx.x];
}

// e^x in FP64 for x <= 0, the exponentials of the FP64 paths (their arguments are
// -2|u| and -u^2/2), after Tang's table method: x = (k / 64) ln2 + r, |r| <= ln2 /
// 128, with ln2 / 64 split into a 32-bit head (so k * head is exact) and the
// rest; e^r from its Taylor series to degree 6 (the remainder is below 3e-20);
// 2^((k mod 64) / 64) from the table; the rest of k is added to the exponent. k
// is the low word of x 64 / ln2 + 1.5 2^52.  Against FP80 over [-700, 0]: at
// most 0.87 ulp off, 1.57 for the series to degree 12 without a table, and
// 12 FP64 instructions for its 18.  Below -707 the result is e^-707 (3e-308);
// the arguments are never positive, infinite or NaN.
__device__ __forceinline__ double exp_nonpos(const double (&tab)[kExpTable], double x) {
  constexpr double kScale = 0x1.71547652b82fep+6;    // 64 / ln 2
  constexpr double kHead = 0x1.62e42feep-7;          // ln 2 / 64 to 32 bits
  constexpr double kRest = 0x1.a39ef35793c76p-39;    // ln 2 / 64 - kHead
  constexpr double kShift = 0x1.8p52;
  x = fmax(x, -707.0);
  const double t = fma(x, kScale, kShift);
  const int k = __double2loint(t);
  const double kd = t - kShift;
  const double r = fma(-kd, kRest, fma(-kd, kHead, x));
  double p = 1.0 / 720.0;
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  const double q = fma(p * r, r, r);
  const double w = tab[k & (kExpTable - 1)];
  const double v = fma(w, q, w);
  return __hiloint2double(__double2hiint(v) + ((k >> 6) << 20), __double2loint(v));
}

// Pointers read from the job table are generic; the hot loops cast row bases
// to the global address space so loads use global_load with a scalar base.
typedef __attribute__((address_space(1))) const char gchar_t;
typedef __attribute__((address_space(1))) const float gfloat_t;
typedef __attribute__((address_space(1))) const double gdouble_t;

__device__ __forceinline__ double lane_of(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

// Reductions within a wave: the lanes of a row of 16 exchange by DPP (a few cycles
// a step, where a shuffle goes through LDS: a lasso path's eight reductions of six
// shuffles took 0.7 us of each join), the four rows' results by readlane.
template <int kCtrl>
__device__ __forceinline__ int dpp(int v) {
  return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xF, 0xF, true);
}
template <int kCtrl>
__device__ __forceinline__ double dpp(double v) {
  return __hiloint2double(dpp<kCtrl>(__double2hiint(v)), dpp<kCtrl>(__double2loint(v)));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;
template <class Op>
__device__ __forceinline__ double wave_reduce(double v, Op op) {
  v = op(v, dpp<kXor1>(v));
  v = op(v, dpp<kXor2>(v));
  v = op(v, dpp<kHalfMirror>(v));
  v = op(v, dpp<kMirror>(v));
  return op(op(lane_of(v, 0), lane_of(v, 16)), op(lane_of(v, 32), lane_of(v, 48)));
}

__device__ __forceinline__ double wave_sum(double v) {
  return wave_reduce(v, [](double a, double b) { return a + b; });
}

// FP64 log cosh and Gaussian-weighted term (marginals and the FP64 pair path).
__device__ inline double logcosh64(double u) {
  const double a = fabs(u);
  return a + log1p(exp(-2.0 * a)) - kLn2;
}
__device__ inline double gauss64(double u) { return u * exp(-0.5 * u * u); }

// The four sums of both residuals of two active positions entirely in FP64 from
// the FP64 residuals (the small-m path and the FP64 decision of near-ties): one
// wave, lanes over samples, of the 64-sample blocks first, first + stride, ...;
// the sums over the lanes are valid in every lane.
// log cosh u = |u| + log(1 + e^{-2|u|}) - ln 2; the logs of a lane's samples
// are taken as the log of their product (each factor is in (1, 2], so 512 of
// them stay below 2^512), one FP64 log per 512 samples.
__device__ inline void pair_sums64(const JobDev& J, int si, int sj, int lane, int first,
                                   int stride, const double (&tab)[kExpTable], double (&v)[4]) {
  double r = J.rho[(int64_t)si * J.d + sj];
  const double lim = 1.0 - kCollinear;
  r = r > lim ? lim : (r < -lim ? -lim : r);
  const double al = 1.0 / sqrt(1.0 - r * r);
  gdouble_t* zi = (gdouble_t*)(J.zd + (int64_t)si * J.ldz);
  gdouble_t* zj = (gdouble_t*)(J.zd + (int64_t)sj * J.ldz);
  const int n = J.n, step = stride * 64;
  double a1 = 0.0, a2 = 0.0, b1 = 0.0, b2 = 0.0;
  double pa = 1.0, pb = 1.0;
  int cnt = 0, tot = 0;
  int s = first * 64 + lane;
  double yi = s < n ? zi[s] : 0.0, yj = s < n ? zj[s] : 0.0;  // fetched one block ahead
  for (; s < n; s += step) {
    const double xi = yi, xj = yj;
    if (s + step < n) {
      yi = zi[s + step];
      yj = zj[s + step];
    }
    const double u = al * (xi - r * xj), w = al * (xj - r * xi);
    const double au = fabs(u), aw = fabs(w);
    a1 += au;
    b1 += aw;
    pa = fma(pa, exp_nonpos(tab, -2.0 * au), pa);
    pb = fma(pb, exp_nonpos(tab, -2.0 * aw), pb);
    a2 += u * exp_nonpos(tab, -0.5 * u * u);
    b2 += w * exp_nonpos(tab, -0.5 * w * w);
    ++tot;
    if (++cnt == 512) {
      a1 += log(pa);
      b1 += log(pb);
      pa = pb = 1.0;
      cnt = 0;
    }
  }
  v[0] = a1 + (log(pa) - (double)tot * kLn2);
  v[1] = a2;
  v[2] = b1 + (log(pb) - (double)tot * kLn2);
  v[3] = b2;
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = wave_sum(v[k]);
}

// R from the sums of pair_sums64 over all samples.
__device__ inline double measure64(const JobDev& J, int si, int sj, const double (&v)[4]) {
  const double inv_n = 1.0 / (double)J.n;
  const double h_ij = entropy_from_moments(v[0] * inv_n, v[1] * inv_n);
  const double h_ji = entropy_from_moments(v[2] * inv_n, v[3] * inv_n);
  return (J.hm[sj] + h_ij) - (J.hm[si] + h_ji);
}


__device__ __forceinline__ float readlane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Block-wide deterministic FP64 sum (256 threads), result valid in all threads.
__device__ double block_sum_256(double v, double* sh) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (tid < off) sh[tid] += sh[tid + off];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// Per-thread sums of the five moments kept for every variable: log cosh z,
// z exp(-z^2/2), z^3, z^4, |z|.  log cosh z = |z| + log(1 + e^{-2|z|}) - ln 2;
// the logs are taken as the log of a running product (each factor in (1, 2],
// flushed every 512 samples), one FP64 log per 512 samples.
// Also what the pair kernels' shared form needs: the largest |z| and the sum
// of the FP32 copies.
struct MomAcc {
  double abs_sum = 0.0, log_sum = 0.0, g = 0.0, z3 = 0.0, z4 = 0.0, prod = 1.0;
  double top = 0.0, copy = 0.0;
  int cnt = 0, tot = 0;
  const double (&tab)[kExpTable];
  __device__ inline explicit MomAcc(const double (&t)[kExpTable]) : tab(t) {}
  __device__ inline double add(double z) {  // returns exp(-z^2 / 2)
    const double a = fabs(z), z2 = z * z;
    const double e = exp_nonpos(tab, -0.5 * z2);
    abs_sum += a;
    top = fmax(top, a);
    copy += (double)(float)z;
    prod *= 1.0 + exp_nonpos(tab, -2.0 * a);
    g += z * e;
    z3 += z2 * z;
    z4 += z2 * z2;
    ++tot;
    if (++cnt == 512) {
      log_sum += log(prod);
      prod = 1.0;
      cnt = 0;
    }
    return e;
  }
  // in the order of store_moments
  __device__ inline void sums(double (&acc)[7]) const {
    acc[0] = abs_sum + (log_sum + log(prod)) - (double)tot * kLn2;
    acc[1] = g;
    acc[2] = z3;
    acc[3] = z4;
    acc[4] = abs_sum;
    acc[kMomTop] = top;
    acc[kMomSum] = copy;
  }
};

// Block-wide deterministic sums (256 threads; of value kMomTop the maximum):
// within waves, then the four wave totals in order.  `sh` holds 28
// doubles.  The result is valid in thread 0.
__device__ inline void block_moments(double (&v)[7], double* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 7; ++k)
    v[k] = k == kMomTop ? wave_reduce(v[k], [](double a, double b) { return fmax(a, b); })
                        : wave_sum(v[k]);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 7; ++k) sh[k * 4 + wave] = v[k];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      const double* w = sh + k * 4;
      v[k] = k == kMomTop ? fmax(fmax(w[0], w[1]), fmax(w[2], w[3]))
                          : ((w[0] + w[1]) + w[2]) + w[3];
    }
}

// Means of the five moments of variable `slot`, its largest |z|, the sum of
// its FP32 copy, and its marginal entropy.
__device__ inline void store_moments(const JobDev& J, int slot, const double (&acc)[7], int n) {
  const double inv = 1.0 / (double)n;
  double* mo = J.mom + (int64_t)slot * 8;
#pragma unroll
  for (int k = 0; k < 5; ++k) mo[k] = acc[k] * inv;
  mo[kMomTop] = acc[kMomTop];
  mo[kMomSum] = acc[kMomSum];
  J.hm[slot] = entropy_from_moments(acc[0] * inv, acc[1] * inv);
}

// A job whose pair kernels may take the shared form: their log2 cosh sums then
// leave out the sum of the (signed) residuals, in units of log2(e), which
// measure_from_sums adds for the whole sample.
__device__ inline bool shared_job(const JobDev& J) { return J.g != nullptr && J.tie_on; }

constexpr double kShareTop = 13.0;  // largest |x| of the shared form's x side

// Largest |z| of active position p (m: padding).
__device__ inline double top_at(const JobDev& J, int m, int p) {
  return p < m ? J.mom[(int64_t)J.act[p] * 8 + kMomTop] : 0.0;
}

// Of the 16 lanes of a 4 x 4 sub-block (lane q: ti of row q / 4, tj of column q % 4):
// both sides hold a variable past kShareTop, so the sub-block's waves took the
// separate form over all samples.  Lanes that do not call it count as below.
__device__ inline bool both_far(double ti, double tj) {
  const uint64_t i = __ballot(!(ti <= kShareTop));
  const uint64_t j = __ballot(!(tj <= kShareTop));
  const int at = threadIdx.x & 48;
  return ((i >> at) & 0xffff) != 0 && ((j >> at) & 0xffff) != 0;
}

// R(si, sj) from the pair kernels' sums over all samples: s[0], s[1] of the
// residual of si on sj, s[2], s[3] of sj on si.  whole: the sums leave nothing
// out (a sub-block of the all-pairs kernel on the diagonal, or both_far).
__device__ inline double measure_from_sums(const JobDev& J, int si, int sj,
                                           const double (&s)[4], bool whole) {
  const double inv_n = 1.0 / (double)J.n;
  double r = J.rho[(int64_t)si * J.d + sj];
  const double lim = 1.0 - kCollinear;
  r = r > lim ? lim : (r < -lim ? -lim : r);
  const double al = 1.0 / sqrt(1.0 - r * r);
  // sums of either residual over the FP32 copies, where they were left out
  const double zi = J.mom[(int64_t)si * 8 + kMomSum], zj = J.mom[(int64_t)sj * 8 + kMomSum];
  const bool left_out = shared_job(J) && !whole;
  const double ui = left_out ? al * (zi - r * zj) : 0.0;
  const double uj = left_out ? al * (zj - r * zi) : 0.0;
  const double h_ij = entropy_from_moments((kLn2 * s[0] + ui) * inv_n, al * s[1] * inv_n);
  const double h_ji = entropy_from_moments((kLn2 * s[2] + uj) * inv_n, al * s[3] * inv_n);
  return (J.hm[sj] + h_ij) - (J.hm[si] + h_ji);
}

// ---------------------------------------------------------------------------
// FP64 MFMA tiles (v_mfma_f64_16x16x4f64): 32 x 32 outputs a workgroup of four
// waves, wave (wi, wj) the 16 x 16 block, 32 values of the contraction a chunk
// ---------------------------------------------------------------------------

typedef double double4_t __attribute__((ext_vector_type(4)));

// Two buffers an operand, [contraction][row or column]; column c of row r lies
// at c ^ swz(r): an MFMA's operand read (16 columns of two rows a half-wave) and
// the transposing writes (4 columns of rows 4 k + u, k < 8) then take every
// bank once, where a padded row of 33 took them two and four times, and those
// LDS cycles, not the MFMAs, were the bound.
struct Tile64 {
  double a[2][32][32], b[2][32][32];
};
__device__ inline int swz(int r) { return (((r >> 2) & 7) << 2) ^ ((r & 1) << 4); }

// acc += A^T B for one chunk of either operand in LDS.
__device__ inline double4_t mfma_block(const double (*a)[32], const double (*b)[32],
                                       double4_t acc) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wi = (wave >> 1) * 16, wj = (wave & 1) * 16;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    const int r = kk * 4 + (lane >> 4), at = (lane & 15) ^ swz(r);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r][wi ^ at], b[r][wj ^ at], acc, 0, 0, 0);
  }
  return acc;
}

// acc += A B over the chunks first .. last - 1.  Thread (lv, ls) = (tid >> 3,
// 4 (tid & 7)) fetches four values of either operand a chunk: la(c, v) fills v
// with A[row lv][ls ..] of chunk c; lb(c, v) with B[ls ..][column lv] (kBT) or
// B[lv][ls ..].  The next chunk is fetched into registers while one is
// multiplied, and LDS holds two, so a chunk costs one barrier and, beyond 8
// MFMAs (64 cycles each), no wait for its own loads.  Covariance of d = 1024,
// n = 8192: 492 us without, 429 with, 259 with the layout of Tile64 too.
template <bool kBT, typename LA, typename LB>
__device__ inline double4_t mfma_chunks(Tile64& T, int first, int last, double4_t acc, LA la,
                                        LB lb) {
  const int lv = threadIdx.x >> 3, ls = (threadIdx.x & 7) * 4;
  double va[4], vb[4];
  if (first < last) {
    la(first, va);
    lb(first, vb);
  }
  for (int c = first, buf = 0; c < last; ++c, buf ^= 1) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int at = lv ^ swz(ls + u);
      T.a[buf][ls + u][at] = va[u];
      if (kBT) T.b[buf][ls + u][at] = vb[u];
      else T.b[buf][lv][(ls + u) ^ swz(lv)] = vb[u];
    }
    __syncthreads();
    if (c + 1 < last) {
      la(c + 1, va);
      lb(c + 1, vb);
    }
    acc = mfma_block(T.a[buf], T.b[buf], acc);
  }
  __syncthreads();  // the buffers may be reused
  return acc;
}

// Four centred samples s .. s + 3 of a row of FP64 (16-byte aligned at s, padded
// past s + 3; zero from n on and for a row that is off).
__device__ inline void centred4(const double* z, int s, int n, bool on, double mu,
                                double (&v)[4]) {
  const double2 lo = *reinterpret_cast<const double2*>(z + s);
  const double2 hi = *reinterpret_cast<const double2*>(z + s + 2);
  v[0] = on && s < n ? lo.x - mu : 0.0;
  v[1] = on && s + 1 < n ? lo.y - mu : 0.0;
  v[2] = on && s + 2 < n ? hi.x - mu : 0.0;
  v[3] = on && s + 3 < n ? hi.y - mu : 0.0;
}

// Register r of a lane's accumulator is D[tile_row(r)][tile_col()].
__device__ inline int tile_row(int r) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave >> 1) * 16 + 4 * r + (lane >> 4);
}
__device__ inline int tile_col() {
  return ((threadIdx.x >> 6) & 1) * 16 + (threadIdx.x & 15);
}

// Partial tiles of a contraction split over workgroups: slot(split, tile) holds
// the 256 threads' four registers; their sum in split order.
__device__ inline void tile_put(double* slot, const double4_t& acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) slot[r * 256 + threadIdx.x] = acc[r];
}
__device__ inline double4_t tile_sum(const double* part, int nsplit, int ntiles, int tile) {
  double4_t acc = {0.0, 0.0, 0.0, 0.0};
  for (int k = 0; k < nsplit; ++k) {
    const double* slot = part + ((int64_t)k * ntiles + tile) * kTileElems + threadIdx.x;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] += slot[r * 256];
  }
  return acc;
}

// Row-major upper-triangular tile index -> (bi, bj), bi <= bj < nb.
__device__ inline void decode_tile(int tile, int nb, int& bi, int& bj) {
  const double B = 2.0 * nb + 1.0;
  int r = (int)((B - sqrt(B * B - 8.0 * (double)tile)) * 0.5);
  r = r < 0 ? 0 : (r > nb - 1 ? nb - 1 : r);
  auto off = [nb](int q) { return q * nb - (q * (q - 1)) / 2; };
  while (r > 0 && off(r) > tile) --r;
  while (r + 1 < nb && off(r + 1) <= tile) ++r;
  bi = r;
  bj = r + (tile - off(r));
}

// ---------------------------------------------------------------------------
// job lookup and schedules
// ---------------------------------------------------------------------------

// Largest j with pre[j] <= b (pre: exclusive prefix sums, pre[njobs] = total);
// that job owns workgroup b and has a non-zero count.
__device__ inline int find_job(const int32_t* __restrict__ pre, int njobs, int b) {
  int lo = 0, hi = njobs;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= b) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Workgroup b belongs to job j at local index b - pre[j]; false when b lies
// beyond the schedule (a grid larger than the device's own totals): the
// workgroup then has nothing to do.
__device__ inline bool locate(const int32_t* __restrict__ pre, int njobs, int b, int& j,
                              int& local) {
  j = find_job(pre, njobs, b);
  local = b - pre[j];
  return local < pre[j + 1] - pre[j];
}

// out[0..njobs] = exclusive prefix sums of count(j); one block of 1024 threads.
template <typename F>
__device__ void block_scan(int njobs, F count, int32_t* out, int32_t* sh) {
  const int tid = threadIdx.x;
  const int per = (njobs + 1023) / 1024;
  const int j0 = tid * per, j1 = min(j0 + per, njobs);
  int32_t s = 0;
  for (int j = j0; j < j1; ++j) s += count(j);
  sh[tid] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int32_t v = tid >= off ? sh[tid - off] : 0;
    __syncthreads();
    sh[tid] += v;
    __syncthreads();
  }
  int32_t run = tid > 0 ? sh[tid - 1] : 0;
  for (int j = j0; j < j1; ++j) {
    out[j] = run;
    run += count(j);
  }
  if (tid == 1023) out[njobs] = sh[1023];
  __syncthreads();
}

struct Best {
  double v;   // measure (NaN mapped to -inf)
  int slot;   // original id
  int pos;    // position in the active list
  double v2;  // runner-up measure
};

__device__ inline bool better(double va, int sa, double vb, int sb) {
  return va > vb || (va == vb && sa < sb);
}

__device__ inline Best merge(const Best& a, const Best& b) {
  Best r;
  if (better(a.v, a.slot, b.v, b.slot)) {
    r = a;
    r.v2 = fmax(a.v2, b.v);
  } else {
    r = b;
    r.v2 = fmax(b.v2, a.v);
  }
  return r;
}

// Grid-stride walk over the workgroup items of a schedule: f(job, local
// index) for items blockIdx.x, blockIdx.x + gridDim.x, ...  (uniform over
// the workgroup, so f may use barriers).
template <typename F>
__device__ __forceinline__ void for_blocks(const int32_t* __restrict__ pre, int njobs, F f) {
  const int total = pre[njobs];
  for (int b = blockIdx.x; b < total; b += gridDim.x) {
    int jb, lb;
    if (!locate(pre, njobs, b, jb, lb)) break;
    f(jb, lb);
  }
}

// for_blocks with neighbouring items on one XCD, so that their rows are shared in
// its L2.
template <typename F>
__device__ __forceinline__ void for_blocks_xcd(const int32_t* __restrict__ pre, int njobs, F f) {
  const int total = pre[njobs];
  for (int b0 = 0; b0 + (int)blockIdx.x < total; b0 += gridDim.x) {
    int jb, lb;
    const int at = xcd_item(blockIdx.x, min((int)gridDim.x, total - b0));
    if (!locate(pre, njobs, b0 + at, jb, lb)) break;
    f(jb, lb);
  }
}

// Pair moments (the hot loop), shared by the all-pairs kernel and the row
// kernels of the learned form.  Grid: per job ntiles * nsplit * (4 / W)
// workgroups of W waves (all pairs: upper-triangular 8 x 8 tiles of positions;
// candidate rows: (K / 8) x nblk tiles whose i side lists candidates).  A
// workgroup owns an 8 x 8 block of (i, j) variables and one range of samples,
// both residual directions of each pair; wave (wi, wj) owns the 4 x 4
// sub-block (i in block bi, j in block bj).  Lanes stride over samples
// (coalesced 256 B loads per variable row).  The wave ends with an FP64
// reduction of every sum over its lanes, stored at
// part[((split * ntiles + tile) * 4 + wave) * 64 + pair * 4 + dir * 2 + which],
// which 0 = S1 (log2 cosh), 1 = S2; dir 0 = residual of i on j, dir 1 = of j
// on i.
//
// Two forms of the sample loop:
//
// Separate (pair_dir, one direction at a time): 7 VALU instructions and 2
// v_exp_f32 an evaluation (see the header).  It holds for any data.  Its sum of
// |u| log2(e) runs over kSumBlock samples at a time, from -kS1Start, so its
// rounding stays that of values below 16.  Its loop takes two blocks a turn: 170
// instructions each, 187 with the next block's rows moved into place.
//
// Shared (pair_both, both directions of a pair at once): 12 VALU and 3
// v_exp_f32 for the two evaluations.
//   * sum log2 cosh u = sum log2(1 + 2^m) - count + log2(e) sum u, m = -2 u
//     log2(e): no |u|, whose sum would cost an instruction.  sum u over all
//     samples follows from the rows' sums, which are kept with the moments (of
//     the FP32 copies: next to 0, but their rounding would otherwise count), so
//     this form leaves it out and measure_from_sums adds it (not for a sub-block
//     with variables past kShareTop on both sides: no wave of it takes this form,
//     and the rows need not be read again for each range's share of the sum, which
//     made 512 x 16384 samples of t4 noise 290 ms for 249).  P = prod
//     (1 + 2^m) is unbounded then: every kRenorm samples its exponent is moved
//     to an integer, which is exact and needs no log in the loop, and a P that
//     has overflowed is noticed there; the wave then measures its range again
//     in the separate form and takes the share of its signed sum out.
//   * u^2 + y^2 = w^2 + x^2 for the residuals u = (x - rho y) alpha and w =
//     (y - rho x) alpha: with E = e^{(x^2 - u^2) / 2} and the stored g = e^{-z^2
//     / 2}, e^{-u^2 / 2} = E g(x) and e^{-w^2 / 2} = E g(y): one exponential
//     for both.  E stays below 2^122 while |x| <= kShareTop.  Past 13.2 in y the
//     stored g(y) is a subnormal, off by at most 2^-150, so E g(y) by 2^-28 =
//     4e-9.  (Subnormals have to be kept, as they are by default: flushed to 0,
//     g(y) would be off by 2^-126 and the weight by up to 0.06.)  So the wave
//     takes as x the side whose four variables stay within kShareTop.
// What bounds both is instruction issue.  Measured on the forms alone, cycles a
// SIMD per evaluation of 64 samples: v_exp_f32 takes 8.2 and lets nothing else
// issue; other FP32 instructions take 4, but down to 2.4 where two waves can
// issue together.  With every wave alternating freely between the two kinds
// they hardly ever do (44 in the separate form, 39 in the shared one).  So the
// arguments, the exponentials and the sums of a pair are kept apart, and a
// wave's exponentials issue at a raised priority: they leave one wave in a run,
// and the others' FP32 instructions meet between the runs (27 in the shared
// form; 38 with the priority on the sums instead; how many pairs share a run
// moves it by 1%).
// FP32 MFMA for the residuals (4x4x1 and 16x16x1 tiles, lanes over pairs)
// keeps VALU instructions from issuing as long as it runs (8 and 32 cycles):
// no gain.  With the rows of the next block loaded while one is evaluated the
// kernel takes 148 registers, three waves a SIMD; without, at four waves, it
// measured the same.  d = 1024, n = 8192: 868 us a launch in the separate form
// (one direction a wave, no priority) to 623 us, 44.7 to 32 cycles.
//
// Without FP64 tie resolution (tie_on 0) every kernel takes the separate
// form, which gives a pair the same bits whatever tile it falls in.  So does a
// job without the g region (a workspace too small for it).  These calls run
// kernels without the shared form (kShared false), a direction a workgroup: four
// waves a SIMD for three, and the others' kernels without the choice, which cost
// k_pair 0.5%.  Order of 1024 x 8192 under fp32_ties: 735 ms (882 before the shared
// form's kernels, 846 in them).
//
// Work items of the pair kernels.  With kLoop false the grid is the schedule
// and workgroup p (after the XCD remap) takes item p.  With kLoop true (gated
// launches whose size the host only bounds) a smaller grid walks the items:
// workgroup p takes items p * chunk .. p * chunk + chunk - 1, chunk =
// ceil(total / G), so a gated-off step costs a few thousand empty workgroups
// instead of the bound.
// Extension mode: the suspect rows against the extension columns only
// (ceil(nsus / 8) x ceil(ne / 8) tiles whose j side lists positions too).
enum PairMode : int { kModeAll = 0, kModeCand = 1, kModeSusp = 2, kModeExt = 3 };

constexpr float kM2 = (float)(-1.0 / (8.0 * kLog2e));  // rounds with relative error 2.7e-9

// Around a run of v_exp_f32: issued at a raised wave priority (see above).
__device__ __forceinline__ void exp_first() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(1);
}
__device__ __forceinline__ void exp_done() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(0);
}

constexpr int kRenorm = 16;         // samples per lane between renormalisations
// most samples per lane of the shared form: the exponents of P and Q share a
// 32-bit register, 16 bits each, and add at most 254 every kRenorm samples
constexpr int kShareMaxIters = 4096;

template <int kMode, int W, bool kShared>
__device__ __forceinline__ void pair_item(const JobDev& J, const JobStep& S, int local, int half,
                                          int wave, int lane);

// W waves per workgroup (1, 2 or 4): every (tile, split) item of item_dirs halves is
// cut into 4 / W consecutive workgroup items a half, and the wave's quadrant of the
// tile is (workgroup item mod 4 / W) * W + its wave in the workgroup.
template <int kMode, bool kLoop, int W, bool kShared>
__device__ __forceinline__ void pair_tiles(const JobDev* __restrict__ jobs, int njobs,
                                           const JobStep* __restrict__ js,
                                           const int32_t* __restrict__ pre, int G) {
  static_assert(W == 1 || W == 2 || W == 4, "1, 2 or 4 waves per workgroup");
  constexpr int kQ = 4 / W;
  const int lane = threadIdx.x & 63;
  const int lw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroups are dispatched round-robin over the 8 XCDs; give every XCD a
  // contiguous range of (job, tile, split) work so that the rows a tile reads
  // are shared in that XCD's L2.
  const int b = blockIdx.x;
  const int p = xcd_item(b, G);
  auto run = [&](int jb, int local) {
    const PairItem it = pair_item_at(local, kQ, kShared);
    pair_item<kMode, W, kShared>(jobs[jb], js[jb], it.item, it.half, it.part * W + lw, lane);
  };
  int jb, local;
  if (!kLoop) {  // the grid is the schedule: one item per workgroup
    if (locate(pre, njobs, p, jb, local)) run(jb, local);
    return;
  }
  const int total = pre[njobs];
  const int chunk = (total + G - 1) / G;
  for (int it = 0; it < chunk; ++it) {
    const int w = p * chunk + it;
    if (w >= total || !locate(pre, njobs, w, jb, local)) break;
    run(jb, local);
  }
}

// One wave's 4 x 4 sub-block over its range of samples.
struct PairWave {
  // coefficients of pair (lane >> 2 & 3, lane & 3) of the sub-block: rho and
  // the scale c1 = -2 log2(e) / sqrt(1 - rho^2).  c1 is not rounded to one
  // FP32 value (that would scale every sample of the pair by the same rounding
  // error and bias its log cosh moment): lanes below n_hi take the FP32 value
  // above c1, the others the one below, so the lanes' mean is c1 to 1/128 of a
  // float spacing and the sample-to-lane assignment carries no bias (a lane's
  // samples are s = lane, lane + 64, ...).
  float r, lo, hi;
  int n_hi;
  int si[4], sj[4];  // variables of either side (d: padding), wave-uniform
  int row;           // variable lane >> 3 of the two sides
  int s_begin, nk;   // first sample, 64-sample blocks
  int lane;
  bool diag;         // both sides hold the same variables
  double* out;       // the wave's 64 partial sums
  float (*lds)[68];  // 32 rows of the wave's own (16-byte aligned, spread banks)
};

// The sums of both moments over the 64 lanes, in FP64, through the wave's own
// LDS block: lane l writes its 32 sums as column l, then lane L adds, in FP64
// and in lane order, sum L & 31 of lanes 32 (L >> 5) .. 32 (L >> 5) + 31, and
// the two halves are added with one exchange; afterwards lane L < 32 holds sum
// L = (a * 4 + c) * 2 + which of the walk (a, c): residual of a on c, a on the
// j side if `transposed` (on a diagonal sub-block direction 1 of pair (c, a)
// where a > c).  `bias` (of that walk index) is added to the log2 cosh sum.  No
// barrier: a wave's LDS operations complete in the order it issues them, and
// no other wave touches the block.
__device__ __forceinline__ void pair_store(const PairWave& w, const float (&A)[16],
                                           const float (&B)[16], double bias, bool transposed,
                                           bool dir1) {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    w.lds[2 * q][w.lane] = A[q];
    w.lds[2 * q + 1][w.lane] = B[q];
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  double v0 = 0.0;
  const float4* row = reinterpret_cast<const float4*>(&w.lds[w.lane & 31][(w.lane >> 5) * 32]);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float4 f = row[j];
    v0 += (double)f.x;
    v0 += (double)f.y;
    v0 += (double)f.z;
    v0 += (double)f.w;
  }
  v0 += __shfl_xor(v0, 32);
  if (w.lane < 32) {
    const int a = w.lane >> 3, c = (w.lane >> 1) & 3, which = w.lane & 1;
    const bool low = w.diag && a > c;
    const int q = (transposed || low) ? c * 4 + a : a * 4 + c;  // i-major pair index
    w.out[q * 4 + ((dir1 || low) ? 2 : 0) + which] = which ? v0 : v0 + bias;
  }
}

// Row bases (wave-uniform) of one side; with a 32-bit per-lane byte offset
// loads use the scalar-base + vector-offset form.
__device__ __forceinline__ void pair_rows(const JobDev& J, const float* base, const int (&s)[4],
                                          gchar_t* (&row)[4]) {
#pragma unroll
  for (int a = 0; a < 4; ++a) row[a] = (gchar_t*)(base + (int64_t)s[a] * J.ldz);
}

// One residual direction of the sub-block, the separate form.  The wave walks
// its 4 x 4 block as (a, c): dir 0 scores residual i|j with i = a, j = c; dir 1
// scores residual j|i with j = a, i = c.  Every lane keeps 64 running values
// (16 pairs x {P, A, S1, S2}).
__device__ __forceinline__ void pair_dir(const JobDev& J, const PairWave& w, int dir) {
  gchar_t *zr[4], *zx[4];  // the regressed variables, the regressors
  pair_rows(J, J.z, dir == 0 ? w.si : w.sj, zr);
  pair_rows(J, J.z, dir == 0 ? w.sj : w.si, zx);
  // each lane lost 1.5 a sample, of which the log2 of the halved cosh accounts
  // for 1
  const double bias = 32.0 * (double)w.nk;
  float kr[16], kc[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int from = dir == 0 ? q : (q & 3) * 4 + (q >> 2);
    kr[q] = readlane_f(w.r, from);
    const float lo = readlane_f(w.lo, from), hi = readlane_f(w.hi, from);
    const int n_hi = __builtin_amdgcn_readlane(w.n_hi, from);
    kc[q] = w.lane < n_hi ? hi : lo;
  }
  float P[16], A[16], S1[16], S2[16];  // A: this block's sum of |u| log2(e)
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    P[q] = 1.f;
    A[q] = -kS1Start;
    S1[q] = S2[q] = 0.f;
  }
  struct Rows {
    float a[4], c[4];
  };
  uint32_t voff = (uint32_t)(w.s_begin + w.lane) * 4u;
  const uint32_t vlast = voff + (uint32_t)(w.nk - 1) * 256u;
  auto load = [&](Rows& x) {  // past the last block: the last one again
    const uint32_t v = voff < vlast ? voff : vlast;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      x.a[a] = *(gfloat_t*)(zr[a] + v);
      x.c[a] = *(gfloat_t*)(zx[a] + v);
    }
    voff += 256u;
  };
  auto eval = [&](const Rows& x) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      float t[4], m1[4], e1[4], e2[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int q = a * 4 + c;
        t[c] = fmaf(-kr[q], x.c[c], x.a[a]);
        m1[c] = kc[q] * fabsf(t[c]);
        e2[c] = (kM2 * m1[c]) * m1[c];
      }
      exp_first();
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        e1[c] = __builtin_amdgcn_exp2f(m1[c]);
        e2[c] = __builtin_amdgcn_exp2f(e2[c]);
      }
      exp_done();
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int q = a * 4 + c;
        P[q] = fmaf(P[q], e1[c], P[q]);
        A[q] = fmaf(m1[c], -0.5f, A[q]);
        S2[q] = fmaf(t[c], e2[c], S2[q]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // two blocks a turn, each loaded while the other is evaluated
  Rows r0, r1;
  load(r0);
  for (int left = w.nk; left > 0; left -= kSumBlock) {
    const int cnt = left < kSumBlock ? left : kSumBlock;
    for (int k = 0; k + 1 < cnt; k += 2) {
      load(r1);
      eval(r0);
      load(r0);
      eval(r1);
    }
    if (cnt & 1) eval(r0);  // the last block of the range (kSumBlock is even)
    const float off = 1.5f * (float)cnt - kS1Start;  // exact
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      S1[q] += (A[q] - off) + __builtin_amdgcn_logf(P[q]);
      P[q] = 1.f;
      A[q] = -kS1Start;
    }
  }
  pair_store(w, S1, S2, bias, dir == 1, dir == 1);
}

// The sums that pair_dir stored made those of the shared form, which leave out the
// signed residuals' share of the range: al (sum of a - rho sum of c) of either
// direction, the eight rows summed in FP64 by eight lanes each.
__device__ __forceinline__ void pair_part(const JobDev& J, const PairWave& w) {
  const float4* z = reinterpret_cast<const float4*>(J.z + (int64_t)w.row * J.ldz + w.s_begin) +
                    (w.lane & 7);
  double v = 0.0;
#pragma unroll 8
  for (int k = 0; k < 2 * w.nk; ++k) {
    const float4 f = z[8 * k];
    v += ((double)f.x + (double)f.y) + ((double)f.z + (double)f.w);
  }
#pragma unroll
  for (int off = 4; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  const int a = (w.lane >> 3) & 3, c = (w.lane >> 1) & 3;  // the walk of pair_store
#pragma unroll
  for (int dir = 0; dir < 2; ++dir) {
    const int q = dir == 0 ? a * 4 + c : c * 4 + a;
    const double sa = __shfl(v, dir == 0 ? a * 8 : 32 + a * 8);
    const double sc = __shfl(v, dir == 0 ? 32 + c * 8 : c * 8);
    // w.lo = -2 log2(e) al to a float's precision
    const double share = 0.5 * (double)__shfl(w.lo, q) * (sa - (double)__shfl(w.r, q) * sc);
    if (w.lane < 32 && (w.lane & 1) == 0) w.out[q * 4 + dir * 2] += share;  // its own store
  }
}

// Both residual directions, the shared form; side 0 takes the i variables as
// x, side 1 the j variables.  False (nothing stored) if a product overflowed.
__device__ __forceinline__ bool pair_both(const JobDev& J, const PairWave& w, int side) {
  constexpr float kX2 = (float)(0.5 * kLog2e);  // rounds with relative error 1.3e-8
  float kr[16], kc[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int from = side == 0 ? q : (q & 3) * 4 + (q >> 2);
    kr[q] = readlane_f(w.r, from);
    const float lo = readlane_f(w.lo, from), hi = readlane_f(w.hi, from);
    const int n_hi = __builtin_amdgcn_readlane(w.n_hi, from);
    kc[q] = w.lane < n_hi ? hi : lo;
  }
  gchar_t *zx[4], *zy[4], *gx[4], *gy[4];
  pair_rows(J, J.z, side == 0 ? w.si : w.sj, zx);
  pair_rows(J, J.z, side == 0 ? w.sj : w.si, zy);
  pair_rows(J, J.g, side == 0 ? w.si : w.sj, gx);
  pair_rows(J, J.g, side == 0 ? w.sj : w.si, gy);
  // u = residual of a (x side) on c: P, S; w = of c on a: Q, T
  float P[16], Q[16], S[16], T[16];
  uint32_t ex[16];  // sums of the biased exponents of P (low half) and Q
  uint32_t top = 0;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    P[q] = Q[q] = 1.f;
    S[q] = T[q] = 0.f;
    ex[q] = 0;
  }
  // the four pairs of variable a at one sample
  auto shared_row = [&](int a, float x, float g, const float (&y)[4], const float (&h)[4]) {
    const float x2 = (kX2 * x) * x;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int q = a * 4 + c;
      const float t = fmaf(-kr[q], y[c], x), v = fmaf(-kr[q], x, y[c]);
      const float mu = kc[q] * t, mw = kc[q] * v, mg = fmaf(kM2 * mu, mu, x2);
      exp_first();
      const float eu = __builtin_amdgcn_exp2f(mu);
      const float ew = __builtin_amdgcn_exp2f(mw);
      const float e = __builtin_amdgcn_exp2f(mg);
      exp_done();
      P[q] = fmaf(P[q], eu, P[q]);
      Q[q] = fmaf(Q[q], ew, Q[q]);
      S[q] = fmaf(t, e * g, S[q]);
      T[q] = fmaf(v, e * h[c], T[q]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  struct Rows {
    float x[4], y[4], gx[4], gy[4];
  };
  uint32_t voff = (uint32_t)(w.s_begin + w.lane) * 4u;
  const uint32_t vlast = voff + (uint32_t)(w.nk - 1) * 256u;
  auto load = [&](Rows& r) {  // past the last block: the last one again
    const uint32_t v = voff < vlast ? voff : vlast;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      r.x[a] = *(gfloat_t*)(zx[a] + v);
      r.y[a] = *(gfloat_t*)(zy[a] + v);
      r.gx[a] = *(gfloat_t*)(gx[a] + v);
      r.gy[a] = *(gfloat_t*)(gy[a] + v);
    }
    voff += 256u;
  };
  auto eval = [&](const Rows& r) {
#pragma unroll
    for (int a = 0; a < 4; ++a) shared_row(a, r.x[a], r.gx[a], r.y, r.gy);
  };
  // two blocks a turn, each loaded while the other is evaluated
  Rows r0, r1;
  load(r0);
  int nf = 0;
  for (int left = w.nk; left > 0; left -= kRenorm, ++nf) {
    const int cnt = left < kRenorm ? left : kRenorm;
    for (int k = 0; k + 1 < cnt; k += 2) {
      load(r1);
      eval(r0);
      load(r0);
      eval(r1);
    }
    if (cnt & 1) eval(r0);  // the last block of the range (kRenorm is even)
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const uint32_t p = __float_as_uint(P[q]), o = __float_as_uint(Q[q]);
      top = max(top, max(p, o));  // both positive: ordered as integers
      ex[q] += ((o >> 23) << 16) + (p >> 23);
      P[q] = __uint_as_float((p & 0x7fffffu) | 0x3f800000u);
      Q[q] = __uint_as_float((o & 0x7fffffu) | 0x3f800000u);
    }
  }
  if (__any(top >= 0x7f800000u)) return false;
  // log2 of each lane's product less 1.5 a sample (its mean is near that, so
  // FP32 holds the difference to 1e-6), put back less the count in FP64
  const int mid = w.nk + (w.nk >> 1);
  const int base = 127 * nf + mid;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    P[q] = (float)((int)(ex[q] & 0xffffu) - base) + __builtin_amdgcn_logf(P[q]);
    Q[q] = (float)((int)(ex[q] >> 16) - base) + __builtin_amdgcn_logf(Q[q]);
  }
  const double bias = 64.0 * (double)(mid - w.nk);
  pair_store(w, P, S, bias, side == 1, side == 1);
  pair_store(w, Q, T, bias, side == 1, side == 0);
  return true;
}

template <int kMode, int W, bool kShared>
__device__ __forceinline__ void pair_item(const JobDev& J, const JobStep& S, int local, int half,
                                          int wave, int lane) {
  constexpr bool kCand = kMode != kModeAll;
  const int m = S.m;
  // sample split: the full step's for all pairs and the extension columns
  const int nsplit = kMode == kModeCand ? S.nsplit_c
                     : kMode == kModeSusp ? S.nsplit_s
                                          : S.nsplit;
  const int ntiles = kMode == kModeAll    ? S.ntiles
                     : kMode == kModeCand ? S.nct
                     : kMode == kModeSusp ? S.nct2
                                          : S.nct3;
  const int split_len = kMode == kModeCand ? S.split_len_c
                        : kMode == kModeSusp ? S.split_len_s
                                             : S.split_len;
  const int tile = local / nsplit, split = local - tile * nsplit;
  int bi, bj;
  if (kCand) {
    const int ncol = kMode == kModeExt ? cdiv(S.ne, kTileVars) : S.nblk;
    bi = tile / ncol;
    bj = tile - bi * ncol;
  } else {
    decode_tile_st(tile, S.nblk, bi, bj);
  }
  const int wi = wave >> 1, wj = wave & 1;
  if (!kCand && bi == bj && wi > wj) return;  // mirror image of quadrant (wj, wi)
  // i side: positions bi * 8 + .. (all pairs) or list entries (candidate /
  // suspect rows; list padding holds position m)
  const int i0 = bi * kTileVars + wi * kWaveVars, pj0 = bj * kTileVars + wj * kWaveVars;
  const int32_t* act = J.act;
  const int32_t* list = kMode == kModeCand ? J.cand : J.cand2;
  auto ipos = [&](int a) { return kCand ? list[i0 + a] : i0 + a; };
  auto jpos = [&](int a) { return kMode == kModeExt ? J.ext[pj0 + a] : pj0 + a; };

  __shared__ __align__(16) float red[W][32][68];
  PairWave w;
  w.lane = lane;
  w.lds = red[threadIdx.x >> 6];
  // opaque: where the compiler knows it to be 0 (the row modes) it merges paths
  // and spills 85 registers
  int diag = !kCand && bi == bj && wi == wj;
  asm("" : "+v"(diag));
  w.diag = __builtin_amdgcn_readfirstlane(diag);
  double* part = kMode == kModeAll ? J.part : (kMode == kModeCand ? J.partc : J.parts);
  w.out = part + (((int64_t)split * ntiles + tile) * 4 + wave) * 64;
  w.s_begin = split * split_len;
  w.nk = (min(w.s_begin + split_len, J.n_pad) - w.s_begin) / 64;
  w.r = w.lo = w.hi = 0.f;
  w.n_hi = 0;
  {
    const int pi = ipos((lane >> 2) & 3), pj = jpos(lane & 3);
    if (pi < m && pj < m && pi != pj) {
      double r = J.rho[(int64_t)act[pi] * J.d + act[pj]];
      const double lim = 1.0 - kCollinear;
      r = r > lim ? lim : (r < -lim ? -lim : r);
      const double c1 = -2.0 * kLog2e * rsqrt(1.0 - r * r);
      w.r = (float)r;
      dither_float(c1, w.lo, w.hi, w.n_hi);
    }
  }
  {
    const int e = (lane >> 3) & 3, p = lane < 32 ? ipos(e) : jpos(e);
    w.row = p < m ? act[p] : J.d;
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {  // wave-uniform: the row bases stay in SGPRs
    w.si[a] = __builtin_amdgcn_readlane(w.row, a * 8);
    w.sj[a] = __builtin_amdgcn_readlane(w.row, 32 + a * 8);
  }
  // A quadrant on the diagonal has the same variables on both sides, so its
  // direction-0 walk (a, c) with a != c already holds both residual
  // directions of each of its 6 pairs.
  if (!kShared) {
    if (half == 0 || !w.diag) pair_dir(J, w, half);
    return;
  }
  bool partial = false;  // the shared form holds, but not over this range
  if (!w.diag) {
    // does either side (i: the lower lanes) reach past kShareTop?  The combining
    // kernels ask the same of the whole sub-block (both_far)
    const double top = w.row < J.d ? J.mom[(int64_t)w.row * 8 + kMomTop] : 0.0;
    const uint64_t far = __ballot(!(top <= kShareTop));
    const int side = (uint32_t)far == 0 ? 0 : (far >> 32 == 0 ? 1 : -1);
    partial = side >= 0;
    if (partial && w.nk <= kShareMaxIters && pair_both(J, w, side)) return;
  }
  const int ndir = w.diag ? 1 : 2;
#pragma clang loop unroll(disable)
  for (int dir = 0; dir < ndir; ++dir) pair_dir(J, w, dir);
  if (partial) pair_part(J, w);
}

}  // namespace
}  // namespace lg
