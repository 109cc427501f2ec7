// gfx950 dense FP64 linear algebra of the library.
//
//   blocked Cholesky     A = L L^T by 32-wide panels, a launch each: the
//                        diagonal block is factored and inverted in one
//                        wave's registers by the workgroup that updated it;
//                        every workgroup multiplies the panel's rows that it
//                        needs by that inverse and gives its 32 x 32 tile of
//                        the trailing lower triangle the rank-32 update, on
//                        FP64 MFMA (16 x 16 x 4).
//   triangular inverse   X = L^-1: the 32 x 32 diagonal blocks, then pairs of
//                        neighbours merged level by level (X21 = -X22 L21
//                        X11, both products on FP64 MFMA), 2 log2(p / 32)
//                        launches.
//   triangular products  op(X) B for the normal equations of the VAR fit:
//                        (L L^T)^-1 C = X^T (X C).
//   covariance           centred Gram matrix of variable rows, permuted into
//                        a given order, on FP64 MFMA.
//   lagged effects       theta_tau = (I - B0) M_tau of VarLiNGAM (Section
//                        3.3: the model's lagged matrices from the VAR ones).
#include "lingam_device.h"
#include "lingam_linalg.h"

namespace lg {
namespace {

constexpr int kNb = 32;  // Cholesky panel width and update tile

typedef double Block[kNb][kNb + 1];

// v[k] -= m col_k for k > j, col_k being lane k's value of col: all lanes are
// read first, so that no product waits for its own, and fenced, or the compiler
// would put every update of a column off to its turn, a chain as long as the
// column's number.
__device__ __forceinline__ void eliminate(double (&v)[32], double m, double col, int j) {
  double s[32];
#pragma unroll
  for (int k = j + 1; k < 32; ++k) s[k] = lane_of(col, k);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = j + 1; k < 32; ++k) v[k] = fma(-m, s[k], v[k]);
  __builtin_amdgcn_sched_barrier(0);
}

// Wave 0 of a workgroup factors the 32 x 32 block in T (lower triangle; rows past
// kb hold the identity) in registers: lane i < 32 holds row i, and column j's
// entries reach the others through readlane.  Lanes 32 + i start from column i
// of the identity: what eliminates column j from the rows, v_k -= v_j L_kj with
// v_j divided by the pivot's root, is the substitution's step for that column,
// so they end with the inverse at no cost.  T holds L, D its inverse on return.
// Bound by the chain of 32 pivots, each a reciprocal root (Newton's iteration
// from v_rsq_f64) and its column's products: 9 us, where elimination in LDS with
// a barrier a column took 17 and the inverse 18 more.  The same with the column
// broadcast out of LDS; loops over the columns in place of code for each: 15 us.
__device__ __forceinline__ void factor_block(Block& T, Block& D, int kb, double tl, Ctrl* ctrl) {
  if (threadIdx.x >= 64) return;
  const int i = threadIdx.x & 31;
  const bool rows = threadIdx.x < 32;
  double v[32];
#pragma unroll
  for (int j = 0; j < 32; ++j) v[j] = rows ? T[i][j] : (i == j ? 1.0 : 0.0);
  bool bad = false;
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    // without a branch: the compiler would move the columns' updates past it
    double piv = lane_of(v[j], j);
    const bool poor = (j < kb) & (!(piv > tl) | !isfinite(piv));
    bad |= poor;
    piv = poor ? 1.0 : piv;
    double y = __builtin_amdgcn_rsq(piv);
    y = fma(0.5 * y, fma(-piv * y, y, 1.0), y);
    y = fma(0.5 * y, fma(-piv * y, y, 1.0), y);
    double root = piv * y;
    root = fma(fma(-root, root, piv), 0.5 * y, root);
    v[j] = rows && i == j ? root : v[j] * y;
    eliminate(v, v[j], v[j], j);
  }
  if (bad && threadIdx.x == 0) set_status(ctrl, kStDegenerate);
#pragma unroll
  for (int j = 0; j < 32; ++j)
    if (rows) T[i][j] = v[j];
    else D[j][i] = v[j];
}

// Factored block and its inverse from LDS to A and X (in full: zeros above the
// diagonal; past kb the block is cut).  Called by every thread of 256.
__device__ __forceinline__ void store_block(Block& T, Block& D, int k0, int kb, double* A,
                                            int64_t lda, double* X, int64_t ldx) {
  for (int e = threadIdx.x; e < kNb * kNb; e += 256) {
    const int i = e >> 5, j = e & 31;
    if (i >= kb || j >= kb) continue;
    if (j <= i) A[(int64_t)(k0 + i) * lda + k0 + j] = T[i][j];
    X[(int64_t)(k0 + i) * ldx + k0 + j] = j <= i ? D[i][j] : 0.0;
  }
}

// Where step k0 finds the columns of its panel, rows below the diagonal block,
// before they are multiplied by its inverse: transposed (row c, column i for
// A[i][k0 + c]), in block rows 0 and 1 of X by turns, right of the diagonal.
__device__ inline double* raw_panel(double* X, int64_t ldx, int k0) {
  return X + (int64_t)(k0 & kNb) * ldx;
}

// tol = 1e-13 * max_j |A_jj| (pivots at or below it are rounding noise) and the
// first diagonal block (workgroup 0); the first panel's columns, 32 rows each
// (the others).
__global__ __launch_bounds__(256) void k_chol_first(double* __restrict__ A, int64_t lda, int p,
                                                    double* __restrict__ X, int64_t ldx,
                                                    double* __restrict__ tol, Ctrl* ctrl,
                                                    size_t wz) {
  __shared__ Block T, D;
  __shared__ double sh[256];
  A = job_at(A, wz);
  X = job_at(X, wz);
  tol = job_at(tol, wz);
  ctrl = job_at(ctrl, wz);
  const int tid = threadIdx.x, kb = p < kNb ? p : kNb, I0 = blockIdx.x * kNb;
  for (int e = tid; e < kNb * kNb; e += 256) {
    const int i = e >> 5, j = e & 31;
    const bool in = I0 + i < p && (I0 > 0 || j <= i);
    T[i][j] = in ? A[(int64_t)(I0 + i) * lda + j] : (i == j ? 1.0 : 0.0);
  }
  if (I0 > 0) {
    __syncthreads();
    for (int e = tid; e < kNb * kNb; e += 256) {
      const int j = e >> 5, i = e & 31;
      if (I0 + i < p) raw_panel(X, ldx, 0)[(int64_t)j * ldx + I0 + i] = T[i][j];
    }
    return;
  }
  double mx = 0.0;
  for (int j = tid; j < p; j += 256) mx = fmax(mx, fabs(A[(int64_t)j * lda + j]));
  sh[tid] = mx;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (tid < off) sh[tid] = fmax(sh[tid], sh[tid + off]);
    __syncthreads();
  }
  const double tl = sh[0] * 1e-13;
  if (tid == 0) tol[0] = tl;
  factor_block(T, D, kb, tl, ctrl);
  __syncthreads();
  store_block(T, D, 0, kb, A, lda, X, ldx);
}

// Step k0 right of its diagonal block (full), r0 = k0 + 32, one 32 x 32 tile
// (I >= J) of the trailing lower triangle per workgroup, on MFMA: the panel's
// rows P_I = A_I L_kk^-T and P_J from the block's inverse (in X), then A_IJ -= P_I
// P_J^T.  Every workgroup forms the rows it needs, which costs it 16 MFMAs a
// wave and saves the launch that would form them first; they are read from
// raw_panel, so those of the first tile column store P_I in place and their tile,
// the next panel, to the next raw_panel; the first workgroup's is the next
// diagonal block, which it factors and inverts.  The product with the inverse
// stands for a solve: against 80-bit arithmetic the panel's error is 1.1 to 1.3 of
// the solve's for 64 x 64 correlation matrices of condition 1e2 to 2e14 (1e-16 to
// 3e-12), the residual 2e-15 of the diagonal for 3e-16.  A launch of 13.8 us a
// step at d = 1024, where a panel solve (32), an update (6) and a factorization with
// a barrier a column (22) were three.
__global__ __launch_bounds__(256) void k_chol_step(double* __restrict__ A, int64_t lda, int p,
                                                   int k0, int nt, double* __restrict__ X,
                                                   int64_t ldx, const double* __restrict__ tol,
                                                   Ctrl* ctrl, size_t wz) {
  __shared__ __align__(16) double PI[32][32], PJ[32][32], Li[32][32];
  __shared__ Block F, D;
  A = job_at(A, wz);
  X = job_at(X, wz);
  tol = job_at(tol, wz);
  ctrl = job_at(ctrl, wz);
  int bj, bi;
  decode_tile(blockIdx.x, nt, bj, bi);  // bj <= bi: tile (I, J) = (bi, bj) is lower
  const int lv = threadIdx.x >> 3, ls = (threadIdx.x & 7) * 4;
  const int r0 = k0 + kNb;
  const int I0 = r0 + bi * kNb, J0 = r0 + bj * kNb;
  const double* raw = raw_panel(X, ldx, k0) + (int64_t)lv * ldx;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = ls + u;
    PI[lv][c ^ swz(lv)] = I0 + c < p ? raw[I0 + c] : 0.0;
    PJ[lv][c ^ swz(lv)] = J0 + c < p ? raw[J0 + c] : 0.0;
    Li[c][lv ^ swz(c)] = X[(int64_t)(k0 + lv) * ldx + k0 + c];
  }
  double4_t t;  // the tile (the diagonal block's past p: identity)
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = I0 + tile_row(r), j = J0 + tile_col();
    t[r] = i < p && j <= i ? A[(int64_t)i * lda + j] : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  const double4_t zero = {0.0, 0.0, 0.0, 0.0};
  const double4_t pi = mfma_block(PI, Li, zero);
  const double4_t pj = bi == bj ? pi : mfma_block(PJ, Li, zero);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = tile_row(r), c = tile_col();
    PI[c][i ^ swz(c)] = pi[r];
    PJ[c][i ^ swz(c)] = pj[r];
    if (bj == 0 && I0 + i < p) A[(int64_t)(I0 + i) * lda + k0 + c] = pi[r];
  }
  __syncthreads();
  t -= mfma_block(PI, PJ, zero);
  if (bj > 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = I0 + tile_row(r), j = J0 + tile_col();
      if (i < p && j <= i) A[(int64_t)i * lda + j] = t[r];
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) F[tile_row(r)][tile_col()] = t[r];
  __syncthreads();
  if (bi > 0) {
    double* next = raw_panel(X, ldx, r0);
    for (int e = threadIdx.x; e < kNb * kNb; e += 256) {
      const int j = e >> 5, i = e & 31;
      if (I0 + i < p) next[(int64_t)j * ldx + I0 + i] = F[i][j];
    }
    return;
  }
  const int kb = min(kNb, p - r0);
  factor_block(F, D, kb, tol[0], ctrl);
  __syncthreads();
  store_block(F, D, r0, kb, A, lda, X, ldx);
}

// Diagonal blocks of X = L^-1 for a unit lower-triangular L, one wave each: lane
// i holds row i of the block and column i of the inverse (the substitution of
// factor_block).
__global__ __launch_bounds__(64) void k_trinv_diag(const double* __restrict__ L, int64_t ldl,
                                                   int p, double* __restrict__ X, int64_t ldx) {
  __shared__ Block T;
  const int I0 = blockIdx.x * kNb, kb = min(kNb, p - I0);
  const int tid = threadIdx.x, i = tid & 31;
  for (int e = tid; e < kNb * kNb; e += 64) {
    const int r = e >> 5, j = e & 31;
    T[r][j] = (r < kb && j < r) ? L[(int64_t)(I0 + r) * ldl + I0 + j] : 0.0;
  }
  __syncthreads();
  double a[32], x[32];
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    a[j] = T[i][j];
    x[j] = i == j ? 1.0 : 0.0;
  }
#pragma unroll
  for (int j = 0; j < 32; ++j) eliminate(x, x[j], a[j], j);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 32; ++r) T[r][i] = x[r];  // both halves of the wave alike
  __syncthreads();
  for (int e = tid; e < kNb * kNb; e += 64) {
    const int r = e >> 5, j = e & 31;
    if (r < kb && j < kb) X[(int64_t)(I0 + r) * ldx + I0 + j] = T[r][j];
  }
}

// One level of X = L^-1: with the diagonal blocks of b rows inverted, those of
// 2 b: [L11 0; L21 L22]^-1 = [X11 0; X21 X22], X21 = -X22 (L21 X11).  A launch
// forms every pair's product L21 X11 (kept transposed in the block of X above
// the diagonal), the next one X21.  log2(p / 32) levels; block row by block
// row it was a chain of p / 32 launches, each as long as its row: d = 1024, 31
// launches of 15.7 us to 10 of 8.  Tiles of all pairs: (b / 32)^2 a pair, the
// last pair's second half cut at p.
__global__ __launch_bounds__(256) void k_trinv_prod(const double* __restrict__ L, int64_t ldl,
                                                    int p, int b, double* __restrict__ X,
                                                    int64_t ldx, size_t wz) {
  __shared__ Tile64 T;
  L = job_at(L, wz);
  X = job_at(X, wz);
  const int nt = b / kNb, pair = blockIdx.x / (nt * nt), e = blockIdx.x - pair * nt * nt;
  const int I = e / nt, J = e - I * nt;
  const int o1 = pair * 2 * b, o2 = o1 + b;  // first rows of the two halves
  if (o2 + I * kNb >= p) return;
  const int lv = threadIdx.x >> 3, ls = (threadIdx.x & 7) * 4;
  const int row = o2 + I * kNb + lv;
  const double4_t acc = mfma_chunks<false>(
      T, J, nt, double4_t{0.0, 0.0, 0.0, 0.0},
      [&](int c, double (&v)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          v[u] = row < p ? L[(int64_t)row * ldl + o1 + c * kNb + ls + u] : 0.0;
      },
      [&](int c, double (&v)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          v[u] = X[(int64_t)(o1 + c * kNb + lv) * ldx + o1 + J * kNb + ls + u];
      });
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = o2 + I * kNb + tile_row(r);
    if (i < p) X[(int64_t)(o1 + J * kNb + tile_col()) * ldx + i] = acc[r];
  }
}

__global__ __launch_bounds__(256) void k_trinv_merge(int p, int b, double* __restrict__ X,
                                                     int64_t ldx, size_t wz) {
  __shared__ Tile64 T;
  X = job_at(X, wz);
  const int nt = b / kNb, pair = blockIdx.x / (nt * nt), e = blockIdx.x - pair * nt * nt;
  const int I = e / nt, J = e - I * nt;
  const int o1 = pair * 2 * b, o2 = o1 + b;
  if (o2 + I * kNb >= p) return;
  const int lv = threadIdx.x >> 3, ls = (threadIdx.x & 7) * 4;
  const int row = o2 + I * kNb + lv;
  const double4_t acc = mfma_chunks<true>(
      T, 0, I + 1, double4_t{0.0, 0.0, 0.0, 0.0},
      [&](int c, double (&v)[4]) {  // X22 (the diagonal block's upper half is zero)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = o2 + c * kNb + ls + u;
          v[u] = row < p && k < p ? X[(int64_t)row * ldx + k] : 0.0;
        }
      },
      [&](int c, double (&v)[4]) {  // the product, transposed above the diagonal
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = o2 + c * kNb + ls + u;
          v[u] = k < p ? X[(int64_t)(o1 + J * kNb + lv) * ldx + k] : 0.0;
        }
      });
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = o2 + I * kNb + tile_row(r);
    if (i < p) X[(int64_t)i * ldx + o1 + J * kNb + tile_col()] = -acc[r];
  }
}

// B[order[i]][order[k]] = -L_ii X_ik for k < i, 0 otherwise (every entry of B
// written once: order is a permutation).
__global__ void k_adj_scatter(const double* __restrict__ L, int64_t ldl,
                              const double* __restrict__ X, int64_t ldx, int p,
                              const int32_t* __restrict__ order, double* __restrict__ B,
                              const Ctrl* ctrl, size_t wz) {
  const int64_t total = (int64_t)p * p;
  if (refused(job_at(ctrl, wz))) return;
  L = job_at(L, wz);
  X = job_at(X, wz);
  order += (int64_t)blockIdx.z * p;
  B += blockIdx.z * total;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / p), k = (int)(e - (int64_t)i * p);
    const double v = k < i ? -L[(int64_t)i * ldl + i] * X[(int64_t)i * ldx + k] : 0.0;
    B[(int64_t)order[i] * p + order[k]] = v;
  }
}

// C = op(A) B for a lower-triangular M x M A (op = A or A^T), B: M x N,
// 32 x 32 output tiles on FP64 MFMA, visiting only the K blocks where op(A)'s
// row block is nonzero.  C must not alias B.
__global__ __launch_bounds__(256) void k_trmm(int M, int N, const double* __restrict__ A,
                                              int64_t lda, int trans, const double* __restrict__ B,
                                              int64_t ldb, double* __restrict__ C, int64_t ldc) {
  __shared__ Tile64 T;
  const int I0 = blockIdx.y * kNb, J0 = blockIdx.x * kNb;
  const int lv = threadIdx.x >> 3, ls = (threadIdx.x & 7) * 4;
  const int cbeg = trans ? blockIdx.y : 0;
  const int cend = trans ? (M + kNb - 1) / kNb : blockIdx.y + 1;
  const double4_t acc = mfma_chunks<false>(
      T, cbeg, cend, double4_t{0.0, 0.0, 0.0, 0.0},
      [&](int c, double (&v)[4]) {  // op(A)[I0 + lv][k]
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = I0 + lv, k = c * kNb + ls + u;
          v[u] = i < M && k < M ? (trans ? A[(int64_t)k * lda + i] : A[(int64_t)i * lda + k]) : 0.0;
        }
      },
      [&](int c, double (&v)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = c * kNb + lv, j = J0 + ls + u;
          v[u] = k < M && j < N ? B[(int64_t)k * ldb + j] : 0.0;
        }
      });
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = I0 + tile_row(r), j = J0 + tile_col();
    if (i < M && j < N) C[(int64_t)i * ldc + j] = acc[r];
  }
}

// S[a][b] = sig[o_a] sig[o_b] rho[o_a][o_b]: a correlation matrix scaled to a
// covariance and permuted into the order o.
__global__ void k_perm_scale(const double* __restrict__ rho, int64_t ldr,
                             const double* __restrict__ sig, const int32_t* __restrict__ order,
                             int d, double* __restrict__ S) {
  const int64_t total = (int64_t)d * d;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int a = (int)(e / d), b = (int)(e - (int64_t)a * d);
    const int oa = order[a], ob = order[b];
    S[e] = sig[oa] * sig[ob] * rho[(int64_t)oa * ldr + ob];
  }
}

// mu[v] = mean of row v of Xd over its first n entries (one workgroup per row).
__global__ __launch_bounds__(256) void k_row_mean(const double* __restrict__ Xd, int64_t ldx, int n,
                                                  double* __restrict__ mu, size_t wz) {
  __shared__ double sh[256];
  Xd = job_at(Xd, wz);
  mu = job_at(mu, wz);
  const double* x = Xd + (int64_t)blockIdx.x * ldx;
  double s = 0.0;
  for (int k = threadIdx.x; k < n; k += 256) s += x[k];
  s = block_sum_256(s, sh);
  if (threadIdx.x == 0) mu[blockIdx.x] = s / (double)n;
}

// S[a][b] = sum_s (x_{o_a}(s) - mu_{o_a}) (x_{o_b}(s) - mu_{o_b}) on FP64 MFMA,
// upper 32 x 32 tiles computed and mirrored; a workgroup per tile and range of
// samples (blockIdx.y), whose tiles k_cov_sum adds when there are several.
__device__ void cov_store(double* S, int d, int bi, int bj, const double4_t& acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = bi * 32 + tile_row(r), j = bj * 32 + tile_col();
    if (i < d && j < d && (bi != bj || i <= j)) {
      S[(int64_t)i * d + j] = acc[r];
      S[(int64_t)j * d + i] = acc[r];
    }
  }
}

__global__ __launch_bounds__(256) void k_cov_perm(const double* __restrict__ Xd, int64_t ldx,
                                                  int n, int d,
                                                  const int32_t* __restrict__ order,
                                                  const double* __restrict__ mu, int nb,
                                                  double* __restrict__ S,
                                                  double* __restrict__ part, const Ctrl* ctrl,
                                                  size_t wz) {
  __shared__ Tile64 T;
  if (refused(job_at(ctrl, wz))) return;
  Xd = job_at(Xd, wz);
  order += (int64_t)blockIdx.z * d;
  mu = job_at(mu, wz);
  S = job_at(S, wz);
  part = job_at(part, wz);
  int bi, bj;
  decode_tile(blockIdx.x, nb, bi, bj);
  const int lv = threadIdx.x >> 3, ls = (threadIdx.x & 7) * 4;
  const int va = bi * 32 + lv < d ? order[bi * 32 + lv] : -1;
  const int vb = bj * 32 + lv < d ? order[bj * 32 + lv] : -1;
  const double* za = Xd + (int64_t)(va < 0 ? 0 : va) * ldx;
  const double* zb = Xd + (int64_t)(vb < 0 ? 0 : vb) * ldx;
  const double ma = va < 0 ? 0.0 : mu[va], mb = vb < 0 ? 0.0 : mu[vb];
  const int chunks = (n + 31) / 32, per = (chunks + gridDim.y - 1) / gridDim.y;
  const double4_t acc = mfma_chunks<true>(
      T, blockIdx.y * per, min((int)(blockIdx.y + 1) * per, chunks), double4_t{0.0, 0.0, 0.0, 0.0},
      [&](int c, double (&v)[4]) { centred4(za, c * 32 + ls, n, va >= 0, ma, v); },
      [&](int c, double (&v)[4]) { centred4(zb, c * 32 + ls, n, vb >= 0, mb, v); });
  if (gridDim.y == 1) cov_store(S, d, bi, bj, acc);
  else tile_put(part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kTileElems, acc);
}

__global__ __launch_bounds__(256) void k_cov_sum(const double* __restrict__ part, int nsplit,
                                                 int d, int nb, double* __restrict__ S,
                                                 size_t wz) {
  part = job_at(part, wz);
  S = job_at(S, wz);
  int bi, bj;
  decode_tile(blockIdx.x, nb, bi, bj);
  cov_store(S, d, bi, bj, tile_sum(part, nsplit, gridDim.x, blockIdx.x));
}

// theta[t][i][j] = M[t][i][j] - sum_k B0[i][k] M[t][k][j] (16 x 16 tiles, LDS).
__global__ __launch_bounds__(256) void k_lagged(const double* __restrict__ M,
                                                const double* __restrict__ B0, int d,
                                                double* __restrict__ theta) {
  __shared__ double Bt[16][17];
  __shared__ double Mt[16][17];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int i = blockIdx.y * 16 + ty, j = blockIdx.x * 16 + tx;
  const double* Mk = M + (int64_t)blockIdx.z * d * d;
  double s = 0.0;
  for (int k0 = 0; k0 < d; k0 += 16) {
    Bt[ty][tx] = (i < d && k0 + tx < d) ? B0[(int64_t)i * d + k0 + tx] : 0.0;
    Mt[ty][tx] = (k0 + ty < d && j < d) ? Mk[(int64_t)(k0 + ty) * d + j] : 0.0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) s += Bt[ty][k] * Mt[k][tx];
    __syncthreads();
  }
  if (i < d && j < d) theta[(int64_t)blockIdx.z * d * d + (int64_t)i * d + j] = Mk[(int64_t)i * d + j] - s;
}

// ---------------------------------------------------------------------------
// adaptive-lasso pruning of the adjacency
// ---------------------------------------------------------------------------

// Xd[v][s] = X[row(s)][v] in FP64 (row(s) = rows[s] or s); padding 0.
__global__ __launch_bounds__(256) void k_gather_f64(const float* __restrict__ X, int64_t ldx,
                                                    const int32_t* __restrict__ rows, int n,
                                                    int d, int n_pad, double* __restrict__ Xd,
                                                    int64_t ldz, Ctrl* ctrl) {
  __shared__ float tile[64][65];
  if (refused(ctrl)) return;
  const int s0 = blockIdx.x * 64, v0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  bool bad = false;
  for (int i = 0; i < 16; ++i) {
    const int sl = ty * 16 + i, s = s0 + sl, v = v0 + tx;
    float val = 0.f;
    if (s < n && v < d) {
      val = X[(int64_t)(rows ? rows[s] : s) * ldx + v];
      bad |= !isfinite(val);
    }
    tile[sl][tx] = val;
  }
  __syncthreads();
  for (int i = 0; i < 16; ++i) {
    const int vl = ty * 16 + i, v = v0 + vl, s = s0 + tx;
    if (v < d && s < n_pad) Xd[(int64_t)v * ldz + s] = (double)tile[tx][vl];
  }
  if (bad) set_status(ctrl, kStDegenerate);
}

// sd[a] = sqrt(S[a][a] / n); R = S scaled to unit diagonal; L = R (to be
// factored), B = 0.  A zero variance sets the status.
__global__ void k_corr(const double* __restrict__ S, int d, int n, double* __restrict__ sd,
                       double* __restrict__ R, double* __restrict__ L, double* __restrict__ B,
                       Ctrl* ctrl) {
  const int64_t total = (int64_t)d * d;
  if (refused(ctrl)) return;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int a = (int)(e / d), b = (int)(e - (int64_t)a * d);
    const double saa = S[(int64_t)a * d + a], sbb = S[(int64_t)b * d + b];
    B[e] = 0.0;
    if (!(saa > 0.0) || !(sbb > 0.0)) {
      set_status(ctrl, kStDegenerate);
      R[e] = L[e] = (a == b) ? 1.0 : 0.0;
    } else {
      const double r = S[e] / sqrt(saa * sbb);
      R[e] = L[e] = r;
    }
    if (a == b) sd[a] = sqrt(fmax(saa, 0.0) / (double)n);
  }
}

// Path state of a target of at most this many predictors in LDS.
constexpr int kLarsLds = 1024;

struct LarsShared {
  // inverse of G on the active set; the refit's matrix with its right side below
  double M[kLassoMaxActive + 1][kLassoMaxActive + 1];
  double g[kLassoMaxActive], v[kLassoMaxActive], wv[kLassoMaxActive], cf[kLassoMaxActive];
  double sgn[kLassoMaxActive];
  int64_t row[kLassoMaxActive];  // idx d: rows of R
  int idx[kLassoMaxActive];
  int best_idx[kLassoMaxActive];
  // the four waves' parts of a reduction, a slot a use, so that one barrier
  // orders it: the next write of a slot lies past other barriers
  double rv[8][4];
  int ri[8][4];
};

// (v, i) against (b, ib): the smaller value, ties to the smaller index; index -1 =
// none.
__device__ __forceinline__ void take_less(double& v, int& i, double b, int ib) {
  const bool less = ib >= 0 && (i < 0 || b < v || (b == v && ib < i));
  v = less ? b : v;
  i = less ? ib : i;
}

// The wave's part of a reduction, left for the workgroup in a slot.
__device__ inline void put_argmin(double v, int i, LarsShared& S, int slot) {
  take_less(v, i, dpp<kXor1>(v), dpp<kXor1>(i));
  take_less(v, i, dpp<kXor2>(v), dpp<kXor2>(i));
  take_less(v, i, dpp<kHalfMirror>(v), dpp<kHalfMirror>(i));
  take_less(v, i, dpp<kMirror>(v), dpp<kMirror>(i));
  double bv = lane_of(v, 0);
  int bi = __builtin_amdgcn_readlane(i, 0);
#pragma unroll
  for (int l = 16; l < 64; l += 16)
    take_less(bv, bi, lane_of(v, l), __builtin_amdgcn_readlane(i, l));
  if ((threadIdx.x & 63) == 0) {
    S.rv[slot][threadIdx.x >> 6] = bv;
    S.ri[slot][threadIdx.x >> 6] = bi;
  }
}
__device__ inline void get_argmin(const LarsShared& S, int slot, double& v, int& i) {
  v = S.rv[slot][0];
  i = S.ri[slot][0];
#pragma unroll
  for (int w = 1; w < 4; ++w) take_less(v, i, S.rv[slot][w], S.ri[slot][w]);
}
__device__ inline void put_sum(double v, LarsShared& S, int slot) {
  v = wave_reduce(v, [](double a, double b) { return a + b; });
  if ((threadIdx.x & 63) == 0) S.rv[slot][threadIdx.x >> 6] = v;
}
__device__ inline double get_sum(const LarsShared& S, int slot) {
  return (S.rv[slot][0] + S.rv[slot][1]) + (S.rv[slot][2] + S.rv[slot][3]);
}
__device__ inline void put_max(double v, LarsShared& S, int slot) {
  v = wave_reduce(v, [](double a, double b) { return fmax(a, b); });
  if ((threadIdx.x & 63) == 0) S.rv[slot][threadIdx.x >> 6] = v;
}
__device__ inline double get_max(const LarsShared& S, int slot) {
  return fmax(fmax(S.rv[slot][0], S.rv[slot][1]), fmax(S.rv[slot][2], S.rv[slot][3]));
}

// sum_{q = c, c + 4, ..} row[q] x[q], q < n <= all, c = tid % 4 (all: the bound of
// the other rows); four products' loads at a time, up to 64 read.
__device__ __forceinline__ double row_dot(const double* row, const double* x, int n, int all) {
  double acc = 0.0;
  for (int q0 = threadIdx.x & 3; q0 < all; q0 += 16) {
    double a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = row[q0 + 4 * u];
      b[u] = x[q0 + 4 * u];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (q0 + 4 * u < n) acc = fma(a[u], b[u], acc);
  }
  return acc;
}

// One workgroup per target position t >= 1 (predictors: positions 0 .. t-1).
// Adaptive weights w_k = |b_k| from the least-squares row of B = I -
// diag(L) L^-1 on the correlation matrix; the lasso path of the weighted
// standardized predictors by least angle regression with the lasso
// modification (covariance form, G_jk = n w_j w_k R_jk, c_k = n w_k R_kt),
// at most max_active active; the breakpoint of least BIC
// n log(2 pi s2) + RSS / s2 + log(n) df, s2 = n L_tt^2 / (n - t - 1); the
// kept predictors refitted by least squares (standardized, then rescaled).
// The inverse of G on the active set lies in LDS, updated by the Schur complement
// on a join and the rank-1 downdate on a leave; so does the path state
// (correlations, coefficients, directions, flags, weights) up to kLarsLds
// predictors, past them in st[t][4][d].  Up to 256, thread k holds predictor k's
// entries of the active rows of R in registers.  A path is a serial chain of up
// to max_active joins and, at d = 200, the only one of its CU, so latency is the
// bound: reductions within waves, one barrier each; products with M by four
// threads a row, in the pass that updates it; six barriers a join.  d = 200, n =
// 5000: 1287 us with trees of barriers, serial sums and the state in memory, 688
// without, 644 with the rows in registers and M passed over once, 575 with DPP.
template <bool kLds, bool kRegs>
__global__ __launch_bounds__(256) void k_lars(const double* __restrict__ R,
                                              const double* __restrict__ L,
                                              const double* __restrict__ Y,
                                              const double* __restrict__ sd,
                                              const int32_t* __restrict__ order, int d, int n,
                                              int cap, double* __restrict__ st,
                                              double* __restrict__ B, Ctrl* ctrl) {
  __shared__ LarsShared S;
  __shared__ double state[kLds ? 6 * kLarsLds : 1];
  if (refused(ctrl)) return;
  const int t = blockIdx.x + 1;
  const int p = t;
  const int tid = threadIdx.x;
  const double nn = (double)n;
  double* corr = kLds ? state : st + (int64_t)t * 4 * d;
  double* beta = corr + (kLds ? kLarsLds : d);
  double* av = beta + (kLds ? kLarsLds : d);
  double* flag = av + (kLds ? kLarsLds : d);
  double* weight = state + (kLds ? 4 * kLarsLds : 0);
  double* with_t = state + (kLds ? 5 * kLarsLds : 0);  // n w_k R_kt
  const double Ltt = L[(int64_t)t * d + t];
  const double* Yt = Y + (int64_t)t * d;
  const double* Rt = R + (int64_t)t * d;  // row t = column t (symmetric)
  auto wgt = [&](int k) { return kLds ? weight[k] : fabs(Ltt * Yt[k]); };
  auto cval = [&](int k) { return kLds ? with_t[k] : nn * wgt(k) * Rt[k]; };
  double x[kRegs ? kLassoMaxActive : 1] = {};  // R[idx_r][tid]
  // inactive predictor of largest |corr| (ties to the smaller position)
  double jv = INFINITY;
  int j = -1;
  for (int k = tid; k < p; k += 256) {
    const double w = fabs(Ltt * Yt[k]), c = nn * w * Rt[k];
    if (kLds) {
      weight[k] = w;
      with_t[k] = c;
    }
    corr[k] = c;
    beta[k] = 0.0;
    flag[k] = 0.0;
    if (-fabs(c) < jv) {
      jv = -fabs(c);
      j = k;
    }
  }
  put_argmin(jv, j, S, 0);
  __syncthreads();
  get_argmin(S, 0, jv, j);
  const double tiny = 1e-14 * fmax(1.0, -jv);
  const double s2 = nn * Ltt * Ltt / (double)(n - p - 1);
  const double logterm = nn * log(2.0 * 3.14159265358979323846 * s2);
  const double lnn = log(nn);
  double best = logterm + nn / s2;  // beta = 0: RSS = n, df = 0
  int best_na = 0;
  int na = 0;
  bool joined = true;
  const int cap_a = cap < p ? cap : p;
  const int max_iter = 8 * kLassoMaxActive + 16;  // bound on the loop (never reached in practice)
  const int r4 = tid >> 2, c4 = tid & 3;  // row of M and first column of this thread
  for (int iter = 0; iter < max_iter; ++iter) {
    double cr = 0.0;  // correlation of active predictor tid
    double ms = 0.0;  // M sgn, row r4
    if (joined) {
      if (na == p) break;
      if (j < 0 || -jv <= tiny) break;
      // Schur complement: append j to the inverse of G on the active set
      const double wj = wgt(j);
      const double* Rj = R + (int64_t)j * d;
      const double Rjj = Rj[j];
      double xj = 0.0;
      if (kRegs && tid < p) xj = Rj[tid];
      if (tid <= na) {
        const int k = tid < na ? S.idx[tid] : j;
        if (tid < na) S.g[tid] = nn * wgt(k) * wj * Rj[k];
        cr = corr[k];
        S.sgn[tid] = cr >= 0.0 ? 1.0 : -1.0;
      }
      __syncthreads();
      double mg = row_dot(S.M[r4], S.g, r4 < na ? na : 0, na);
      mg += dpp<kXor1>(mg);
      mg += dpp<kXor2>(mg);
      const bool own = r4 < na && c4 == 0;
      if (own) S.v[r4] = mg;
      put_sum(own ? S.g[r4] * mg : 0.0, S, 1);
      put_max(fabs(cr), S, 3);
      if (tid == 0) {
        S.idx[na] = j;
        S.row[na] = (int64_t)j * d;
        flag[j] = 1.0;
      }
      __syncthreads();
      const double sch = nn * wj * wj * Rjj - get_sum(S, 1);
      if (!(sch > 1e-12 * nn * wj * wj)) break;  // the new predictor is (nearly) collinear
      // M and, in the same pass, its product with the signs
      const double rs = 1.0 / sch, vr = r4 < na ? mg * rs : -rs;
      for (int q0 = c4; q0 <= na; q0 += 16) {
        double m[4], v[4], sg[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          m[u] = S.M[r4][q0 + 4 * u];
          v[u] = S.v[q0 + 4 * u];
          sg[u] = S.sgn[q0 + 4 * u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = q0 + 4 * u;  // row and column na: -v / sch, 1 / sch
          const double e = fma(q < na ? v[u] : -1.0, vr, r4 < na && q < na ? m[u] : 0.0);
          if (r4 <= na && q <= na) {
            S.M[r4][q] = e;
            ms = fma(e, sg[u], ms);
          }
        }
      }
      if (kRegs) {
#pragma unroll
        for (int r = 0; r < kLassoMaxActive; ++r) x[r] = r == na ? xj : x[r];
      }
      ++na;
    } else {
      if (tid < na) {
        cr = corr[S.idx[tid]];
        S.sgn[tid] = cr >= 0.0 ? 1.0 : -1.0;
      }
      put_max(fabs(cr), S, 3);
      __syncthreads();
      ms = row_dot(S.M[r4], S.sgn, r4 < na ? na : 0, na);
    }
    // equiangular direction on the active set
    ms += dpp<kXor1>(ms);
    ms += dpp<kXor2>(ms);
    const bool own = r4 < na && c4 == 0;
    put_sum(own ? S.sgn[r4] * ms : 0.0, S, 2);
    __syncthreads();
    const double AA = 1.0 / sqrt(get_sum(S, 2));
    const double C = get_max(S, 3);
    if (c4 == 0) {
      S.wv[r4] = r4 < na ? AA * ms : 0.0;
      S.cf[r4] = r4 < na ? nn * wgt(S.idx[r4]) * (AA * ms) : 0.0;
    }
    __syncthreads();
    // a_k = sum_r G(k, idx_r) wv_r, and the first join along the direction
    double gj = INFINITY;
    int kj = -1;
    for (int k = tid; k < p; k += 256) {
      double acc = 0.0;
      if (kRegs) {
#pragma unroll
        for (int r0 = 0; r0 < kLassoMaxActive; r0 += 16)
          if (r0 < na)
#pragma unroll
            for (int u = 0; u < 16; ++u) acc = fma(S.cf[r0 + u], x[r0 + u], acc);  // cf 0 past na
      } else {
        for (int r0 = 0; r0 < na; r0 += 16) {  // rows past the last: read again, times 0
          double y[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) y[u] = R[S.row[min(r0 + u, na - 1)] + k];
#pragma unroll
          for (int u = 0; u < 16; ++u)
            if (r0 + u < na) acc = fma(S.cf[r0 + u], y[u], acc);
        }
      }
      acc *= wgt(k);
      av[k] = acc;
      if (flag[k] == 0.0) {
        const double ck = corr[k];
        const double d1 = AA - acc, d2 = AA + acc;
        if (d1 > 0.0) {
          const double g = (C - ck) / d1;
          if (g > 0.0 && g < gj) {
            gj = g;
            kj = k;
          }
        }
        if (d2 > 0.0) {
          const double g = (C + ck) / d2;
          if (g > 0.0 && g < gj) {
            gj = g;
            kj = k;
          }
        }
      }
    }
    // first active coefficient to reach zero
    double gl = INFINITY;
    int rl = -1;
    if (tid < na && S.wv[tid] != 0.0) {
      const double g = -beta[S.idx[tid]] / S.wv[tid];
      if (g > 0.0) {
        gl = g;
        rl = tid;
      }
    }
    put_argmin(gj, kj, S, 4);
    put_argmin(gl, rl, S, 5);
    __syncthreads();
    double gjoin, gleave;
    int jn, lr;
    get_argmin(S, 4, gjoin, jn);
    get_argmin(S, 5, gleave, lr);
    double gam = C / AA;
    int event = 0;  // 0 end, 1 join, 2 leave
    if (jn >= 0 && gjoin < gam) {
      gam = gjoin;
      event = 1;
    }
    if (lr >= 0 && gleave < gam) {
      gam = gleave;
      event = 2;
    }
    // step; the criterion at the new breakpoint: RSS = n - beta'c - beta'corr
    double part = 0.0;
    if (tid < na) {
      const int k = S.idx[tid];
      const double bk = beta[k] + gam * S.wv[tid];
      beta[k] = bk;
      if (event != 2 || tid != lr) part = bk * (cval(k) + (cr - gam * av[k]));
    }
    jv = INFINITY;
    j = -1;
    for (int k = tid; k < p; k += 256) {
      const double c = corr[k] - gam * av[k];
      corr[k] = c;
      if (flag[k] == 0.0 && -fabs(c) < jv) {
        jv = -fabs(c);
        j = k;
      }
    }
    put_argmin(jv, j, S, 6);  // who joins next
    put_sum(part, S, 7);
    __syncthreads();
    get_argmin(S, 6, jv, j);
    const double bsum = get_sum(S, 7);
    if (event == 2) {
      const int who = S.idx[lr];
      // rank-1 downdate of the inverse without row / column lr, then compaction
      const double piv = S.M[lr][lr];
      double keep[16];
      const int nb = na - 1;
      int cnt = 0;
      for (int e = tid; e < nb * nb; e += 256, ++cnt) {
        const int r2 = e / nb, q2 = e - r2 * nb;
        const int r = r2 + (r2 >= lr ? 1 : 0), q = q2 + (q2 >= lr ? 1 : 0);
        keep[cnt] = S.M[r][q] - S.M[r][lr] * S.M[lr][q] / piv;
      }
      int idx_keep = tid < nb ? S.idx[tid + (tid >= lr ? 1 : 0)] : 0;
      __syncthreads();
      cnt = 0;
      for (int e = tid; e < nb * nb; e += 256, ++cnt) {
        const int r2 = e / nb, q2 = e - r2 * nb;
        S.M[r2][q2] = keep[cnt];
      }
      if (tid < nb) {
        S.idx[tid] = idx_keep;
        S.row[tid] = (int64_t)idx_keep * d;
      }
      if (kRegs) {
#pragma unroll
        for (int r = 0; r + 1 < kLassoMaxActive; ++r) x[r] = r >= lr ? x[r + 1] : x[r];
      }
      if (tid == 0) {
        beta[who] = 0.0;
        flag[who] = 0.0;
      }
      __syncthreads();
      na = nb;
    }
    const double crit = logterm + (nn - bsum) / s2 + lnn * (double)na;
    if (crit < best) {
      best = crit;
      best_na = na;
      if (tid < na) S.best_idx[tid] = S.idx[tid];
    }
    if (event == 0) break;
    if (event == 1 && na >= cap_a) break;
    joined = event == 1;
  }
  __syncthreads();
  // refit the kept predictors by least squares on the standardized data
  const int ns = best_na;
  if (ns == 0) return;
  for (int e = tid; e < ns * ns; e += 256) {
    const int r = e / ns, q = e - r * ns;
    S.M[r][q] = R[(int64_t)S.best_idx[r] * d + S.best_idx[q]];
  }
  if (tid < ns) S.M[ns][tid] = Rt[S.best_idx[tid]];  // row ns ends as L^-1 of it
  __syncthreads();
  for (int j = 0; j < ns; ++j) {  // Cholesky in LDS, lower triangle
    double a = S.M[j][j];
    if (!(a > 1e-13)) {
      if (tid == 0) set_status(ctrl, kStDegenerate);
      a = 1.0;
    }
    const double root = sqrt(a);
    if (tid > j && tid <= ns) S.M[tid][j] /= root;
    __syncthreads();
    if (tid == j) S.M[j][j] = root;
    const int w = ns - j;  // rows j + 1 .. ns, columns up to ns - 1
    for (int e = tid; e < w * w; e += 256) {
      const int ii = e / w, kk = e - ii * w;
      if (kk <= ii && kk < w - 1)
        S.M[j + 1 + ii][j + 1 + kk] -= S.M[j + 1 + ii][j] * S.M[j + 1 + kk][j];
    }
    __syncthreads();
  }
  if (tid >= 64) return;
  double z = tid < ns ? S.M[ns][tid] : 0.0;  // backward substitution, lane i unknown i
  for (int i = ns - 1; i >= 0; --i) {
    const double x = __shfl(z, i) / S.M[i][i];
    if (tid == i) z = x;
    else if (tid < i) z -= S.M[i][tid] * x;
  }
  if (tid < ns) {
    const int k = S.best_idx[tid];
    B[(int64_t)order[t] * d + order[k]] = z * sd[t] / sd[k];
  }
}

// A[a][b] = 1 (a == b), -B[o_a][o_b] (a > b), 0 (a < b): I - B in the causal
// order, unit lower triangular (entries of B above that triangle ignored).
__global__ void k_unit_lower(const double* __restrict__ B, const int32_t* __restrict__ order,
                             int d, double* __restrict__ A) {
  const int64_t total = (int64_t)d * d;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int a = (int)(e / d), b = (int)(e - (int64_t)a * d);
    A[e] = a == b ? 1.0 : (a > b ? -B[(int64_t)order[a] * d + order[b]] : 0.0);
  }
}

// T[o_a][o_b] = X[a][b] for a >= b, 0 otherwise (every entry written once).
__global__ void k_scatter_lower(const double* __restrict__ X, const int32_t* __restrict__ order,
                                int d, double* __restrict__ T) {
  const int64_t total = (int64_t)d * d;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int a = (int)(e / d), b = (int)(e - (int64_t)a * d);
    T[(int64_t)order[a] * d + order[b]] = a >= b ? X[e] : 0.0;
  }
}

unsigned grid_for(int64_t n) {
  const int64_t g = (n + 255) / 256;
  return (unsigned)(g < 4096 ? (g < 1 ? 1 : g) : 4096);
}

}  // namespace

// X's blocks below the diagonal from its diagonal blocks, level by level.
static hipError_t tri_levels(const double* L, int64_t ldl, int p, double* X, int64_t ldx,
                             int count, size_t wz, hipStream_t st) {
  for (int b = kNb; b < p; b *= 2) {
    const int nt = b / kNb, pairs = (p - b + 2 * b - 1) / (2 * b);
    const dim3 g((unsigned)(pairs * nt * nt), 1, (unsigned)count);
    hipLaunchKernelGGL(k_trinv_prod, g, dim3(256), 0, st, L, ldl, p, b, X, ldx, wz);
    hipLaunchKernelGGL(k_trinv_merge, g, dim3(256), 0, st, p, b, X, ldx, wz);
  }
  return hipGetLastError();
}

hipError_t launch_cholesky_inverse(double* A, int64_t lda, int p, double* X, int64_t ldx,
                                   double* tol, Ctrl* ctrl, int count, size_t wz,
                                   hipStream_t st) {
  const unsigned z = (unsigned)count;
  hipLaunchKernelGGL(k_chol_first, dim3((unsigned)((p + kNb - 1) / kNb), 1, z), dim3(256), 0, st,
                     A, lda, p, X, ldx, tol, ctrl, wz);
  for (int k0 = 0; k0 + kNb < p; k0 += kNb) {
    const int nt = (p - k0 - 1) / kNb;  // blocks of rows below the diagonal block
    hipLaunchKernelGGL(k_chol_step, dim3((unsigned)(nt * (nt + 1) / 2), 1, z), dim3(256), 0, st,
                       A, lda, p, k0, nt, X, ldx, (const double*)tol, ctrl, wz);
  }
  return tri_levels(A, lda, p, X, ldx, count, wz, st);
}

hipError_t launch_unit_inverse(const double* L, int64_t ldl, int p, double* X, int64_t ldx,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_trinv_diag, dim3((unsigned)((p + kNb - 1) / kNb)), dim3(64), 0, st, L, ldl,
                     p, X, ldx);
  return tri_levels(L, ldl, p, X, ldx, 1, 0, st);
}

hipError_t launch_tri_adjacency(double* A, int p, const int32_t* order, double* B, double* Y,
                                double* tol, Ctrl* ctrl, int count, size_t wz, hipStream_t st) {
  LG_HIP(launch_cholesky_inverse(A, p, p, Y, p, tol, ctrl, count, wz, st));
  hipLaunchKernelGGL(k_adj_scatter, dim3(grid_for((int64_t)p * p), 1, (unsigned)count), dim3(256),
                     0, st, (const double*)A, (int64_t)p, Y, (int64_t)p, p, order, B,
                     (const Ctrl*)ctrl, wz);
  return hipGetLastError();
}

hipError_t launch_trmm(int M, int N, const double* A, int64_t lda, bool trans, const double* B,
                       int64_t ldb, double* C, int64_t ldc, hipStream_t st) {
  dim3 g((unsigned)((N + kNb - 1) / kNb), (unsigned)((M + kNb - 1) / kNb));
  hipLaunchKernelGGL(k_trmm, g, dim3(256), 0, st, M, N, A, lda, trans ? 1 : 0, B, ldb, C, ldc);
  return hipGetLastError();
}

hipError_t launch_perm_scale(const double* rho, int64_t ldr, const double* sig,
                             const int32_t* order, int d, double* S, hipStream_t st) {
  hipLaunchKernelGGL(k_perm_scale, dim3(grid_for((int64_t)d * d)), dim3(256), 0, st, rho, ldr,
                     sig, order, d, S);
  return hipGetLastError();
}

hipError_t launch_cov_perm(const double* Xd, int64_t ldx, int n, int d, const int32_t* order,
                           double* mu, double* S, int nsplit, double* part, const Ctrl* ctrl,
                           int count, size_t wz, hipStream_t st) {
  const unsigned z = (unsigned)count;
  hipLaunchKernelGGL(k_row_mean, dim3((unsigned)d, 1, z), dim3(256), 0, st, Xd, ldx, n, mu, wz);
  const int nb = (d + 31) / 32;
  const unsigned tiles = (unsigned)(nb * (nb + 1) / 2);
  hipLaunchKernelGGL(k_cov_perm, dim3(tiles, (unsigned)nsplit, z), dim3(256), 0, st, Xd, ldx, n,
                     d, order, (const double*)mu, nb, S, part, ctrl, wz);
  if (nsplit > 1)
    hipLaunchKernelGGL(k_cov_sum, dim3(tiles, 1, z), dim3(256), 0, st, (const double*)part, nsplit,
                       d, nb, S, wz);
  return hipGetLastError();
}

hipError_t launch_lagged_effects(const double* M, const double* B0, int d, int lags,
                                 double* theta, hipStream_t st) {
  const unsigned g = (unsigned)((d + 15) / 16);
  hipLaunchKernelGGL(k_lagged, dim3(g, g, (unsigned)lags), dim3(256), 0, st, M, B0, d, theta);
  return hipGetLastError();
}

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

PruneLayout make_prune_layout(int64_t n, int64_t d) {
  PruneLayout A{};
  A.n = n;
  A.d = d;
  A.ldx = (n + 63) / 64 * 64;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  const size_t dd = sizeof(double) * (size_t)d * (size_t)d;
  A.ctrl = take(sizeof(Ctrl));
  A.mark = take(sizeof(int32_t) * (size_t)d);
  A.tol = take(sizeof(double));
  A.mu = take(sizeof(double) * (size_t)d);
  A.sd = take(sizeof(double) * (size_t)d);
  A.xd = take(sizeof(double) * (size_t)d * (size_t)A.ldx);
  A.s = take(dd);
  A.r = take(dd);
  A.l = take(dd);
  A.y = take(dd);
  A.st = take(4 * dd);
  A.total = off;
  return A;
}

hipError_t launch_adjacency_pruned(const PruneLayout& A, char* ws, const float* X, int64_t ldx,
                                   const int32_t* rows, const int32_t* order, int max_active,
                                   double* B, hipStream_t st) {
  Ctrl* ctrl = at<Ctrl>(ws, A.ctrl);
  double* Xd = at<double>(ws, A.xd);
  double* Sm = at<double>(ws, A.s);
  double* Rm = at<double>(ws, A.r);
  double* Lm = at<double>(ws, A.l);
  double* Ym = at<double>(ws, A.y);
  const int d = (int)A.d, n = (int)A.n;
  dim3 g1((unsigned)(A.ldx / 64), (unsigned)((A.d + 63) / 64));
  hipLaunchKernelGGL(k_gather_f64, g1, dim3(256), 0, st, X, ldx, rows, n, d, (int)A.ldx, Xd,
                     A.ldx, ctrl);
  // partial tiles lie in the regions from the correlation matrix on (7 d^2
  // doubles), which are written later
  LG_HIP(launch_cov_perm(Xd, A.ldx, n, d, order, at<double>(ws, A.mu), Sm,
                         gram_splits(n, d, 7 * (int64_t)d * d / kTileElems), Rm, ctrl, 1, 0, st));
  const int64_t dd = (int64_t)d * d;
  hipLaunchKernelGGL(k_corr, dim3(grid_for(dd)), dim3(256), 0, st, (const double*)Sm, d, n,
                     at<double>(ws, A.sd), Rm, Lm, B, ctrl);
  LG_HIP(launch_cholesky_inverse(Lm, d, d, Ym, d, at<double>(ws, A.tol), ctrl, 1, 0, st));
  if (d < 2) return hipGetLastError();
  const int cap = max_active < kLassoMaxActive ? max_active : kLassoMaxActive;
  // a thread a predictor: its rows' entries fit in registers; the path state in LDS
  // (1024: 48 KB beside the inverse's 34, two workgroups a CU, as registers allow)
  const auto lars = d - 1 <= 256        ? k_lars<true, true>
                    : d - 1 <= kLarsLds ? k_lars<true, false>
                                        : k_lars<false, false>;
  hipLaunchKernelGGL(lars, dim3((unsigned)(d - 1)), dim3(256), 0, st, (const double*)Rm,
                     (const double*)Lm, (const double*)Ym, (const double*)at<double>(ws, A.sd),
                     order, d, n, cap, at<double>(ws, A.st), B, ctrl);
  return hipGetLastError();
}

EffectsLayout make_effects_layout(int64_t d) {
  EffectsLayout A{};
  A.d = d;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  A.ctrl = take(sizeof(Ctrl));
  A.mark = take(sizeof(int32_t) * (size_t)d);
  A.a = take(sizeof(double) * (size_t)d * (size_t)d);
  A.x = take(sizeof(double) * (size_t)d * (size_t)d);
  A.total = off;
  return A;
}

hipError_t launch_total_effects(const EffectsLayout& A, char* ws, const double* B,
                                const int32_t* order, double* T, hipStream_t st) {
  const int d = (int)A.d;
  const int64_t dd = (int64_t)d * d;
  double* Am = at<double>(ws, A.a);
  double* Xm = at<double>(ws, A.x);
  hipLaunchKernelGGL(k_unit_lower, dim3(grid_for(dd)), dim3(256), 0, st, B, order, d, Am);
  LG_HIP(launch_unit_inverse(Am, d, d, Xm, d, st));
  hipLaunchKernelGGL(k_scatter_lower, dim3(grid_for(dd)), dim3(256), 0, st, (const double*)Xm,
                     order, d, T);
  return hipGetLastError();
}

}  // namespace lg
