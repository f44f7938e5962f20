// Truncated SVD pseudoinverse of a strongly graded matrix (the periodizing
// matrix Q of Sec. 4.2, whose spherical-harmonic columns decay like
// j_l(k r) over twenty orders of magnitude), organised so that one-sided
// Jacobi runs on a small, well-preconditioned factor:
//
//  1. columns with norm below 1e-15 of the largest are set aside (their
//     coefficients are zero; the perturbation is below the SVD's own
//     rounding level eps*sqrt(n)*s_max), and the rest are ordered by
//     decreasing norm;
//  2. blocked Householder QR without pivoting of the ordered columns,
//     Q P = Q_1 R_1, which takes the tall matrix (2304 rows for a half of the
//     k = 10 periodizer) down to its n2 x n2 triangle with matrix-product
//     work; a column-pivoted Householder QR of that triangle, R_1 P_2 = Q_2 R;
//     trailing rows of R whose joint Frobenius norm is below 1e-15 of the
//     largest column norm are dropped: ~ R_top (r x n2);
//  3. LQ of R_top via QR of R_top^H = Z L^H;
//  4. one-sided Jacobi SVD of the r x r factor L = U_L S V_L^H, truncated at
//     rel_cutoff * s_max as in the paper;
//  5. Q^+ = P P_2 (Z V_L S^{-1}) (Q_1 Q_2 [U_L; 0])^H, V_L S^{-1} = L^{-1} U_L:
//     U and W = P P_2 Z V_L S^{-1} are formed explicitly for the two-stage apply.
// Ordering, pivoting and LQ are the preconditioning that makes one-sided
// Jacobi converge in a handful of sweeps, and the pivoted triangle's graded rows
// are what L^{-1} U_L rests on (svd.hip).  The result is the truncated
// pseudoinverse the paper prescribes, to rounding.
#include <algorithm>
#include <cmath>

#include <string>
#include <thread>

#include "gpinv.hpp"

namespace mfs {

void qr_form_u(const MatDesc *descs, const std::vector<MatDesc> &h, int maxrank, hipStream_t s,
               bool from_identity = false, int nb = kQRNB);
void launch_zero(double2 *p, long n, hipStream_t s);
// halves: matrices 2 i and 2 i + 1 share the cutoff's scale
void jac_sort(const MatDesc *descs, const std::vector<MatDesc> &h, double rel_cutoff, hipStream_t s,
              std::vector<int> &ranks, bool halves = false);
void qrcp_blocked(const MatDesc *descs, const std::vector<MatDesc> &h, double *norms, int *piv, int ld,
                  hipStream_t s);

namespace {

__global__ __launch_bounds__(256) void colnorm_kernel(const MatDesc *__restrict__ d, double *out, int ld) {
  const MatDesc m = d[blockIdx.y];
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (c >= m.n) return;
  const double2 *a = m.a + (size_t)c * m.lda;
  double s = 0.0;
  for (int r = lane; r < m.m; r += 64) s += cabs2(a[r]);
  s = wave_sum(s);
  if (lane == 0) out[(size_t)blockIdx.y * ld + c] = sqrt(s);
}

// dst column i = src column perm[i], times scale[perm[i]] when scale is given;
// only the matrices with only[w] != 0 when that is given
__global__ void gather_kernel(const MatDesc *__restrict__ src, const MatDesc *__restrict__ dst,
                              const int *__restrict__ perm, int ldp, const double *__restrict__ scale,
                              const int *__restrict__ only) {
  if (only && !only[blockIdx.y]) return;
  const MatDesc s = src[blockIdx.y], d = dst[blockIdx.y];
  const int i = blockIdx.x;
  if (i >= d.n) return;
  const int c = perm[(size_t)blockIdx.y * ldp + i];
  const double f = scale ? scale[(size_t)blockIdx.y * ldp + c] : 1.0;
  for (int r = threadIdx.x; r < d.m; r += blockDim.x) d.a[(size_t)i * d.lda + r] = cscale(s.a[(size_t)c * s.lda + r], f);
}

// y = R x, R = triu(a[0:n, 0:n]) (thread per row; a column's rows are
// contiguous, so each step over j is one coalesced read)
__global__ void trimv_kernel(const MatDesc *__restrict__ d, const double2 *__restrict__ x,
                             double2 *__restrict__ y, int ld) {
  const MatDesc m = d[blockIdx.y];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int j0 = blockIdx.x * blockDim.x;
  if (j0 >= m.n) return;
  const double2 *xw = x + (size_t)blockIdx.y * ld;
  double2 acc = cz(0.0, 0.0);
  for (int j = j0; j < m.n; ++j)
    if (i < m.n && j >= i) cfma(acc, m.a[(size_t)j * m.lda + i], xw[j]);
  if (i < m.n) y[(size_t)blockIdx.y * ld + i] = acc;
}

// z = R^H y (one wave per column j: sum over rows i <= j of conj(R_ij) y_i)
__global__ __launch_bounds__(256) void trimhv_kernel(const MatDesc *__restrict__ d, const double2 *__restrict__ y,
                                                     double2 *__restrict__ z, int ld) {
  const MatDesc m = d[blockIdx.y];
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (j >= m.n) return;
  const double2 *yw = y + (size_t)blockIdx.y * ld;
  double2 acc = cz(0.0, 0.0);
  for (int i = lane; i <= j; i += 64) cfmac(acc, m.a[(size_t)j * m.lda + i], yw[i]);
  acc = wave_sum(acc);
  if (lane == 0) z[(size_t)blockIdx.y * ld + j] = acc;
}

// Complete orthogonal decomposition: U_L = I and L^{-1} = (R_L^{-1})^H in
// place of the Jacobi's U_L and V_L S^+ (x: R_L^{-1}, upper triangular)
__global__ void cod_prep_kernel(const MatDesc *__restrict__ qd, const MatDesc *__restrict__ ld,
                                const MatDesc *__restrict__ xd) {
  const MatDesc q = qd[blockIdx.y], l = ld[blockIdx.y], x = xd[blockIdx.y];
  const int k = blockIdx.x;
  const int r = l.n;
  if (k >= r) return;
  double2 *uq = q.u + (size_t)k * q.lda;
  double2 *ul = l.u + (size_t)k * l.lda;
  for (int i = threadIdx.x; i < q.m; i += blockDim.x) uq[i] = cz(i == k ? 1.0 : 0.0, 0.0);
  for (int i = threadIdx.x; i < l.m; i += blockDim.x)
    ul[i] = (i >= k && i < r) ? cconj(x.a[(size_t)i * x.lda + k]) : cz(0.0, 0.0);
}

// squared norms of the rows of R = triu(a[0:n, 0:n])
__global__ void rownorm_kernel(const MatDesc *__restrict__ d, double *out, int ld) {
  const MatDesc m = d[blockIdx.y];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m.n) return;
  double s = 0.0;
  for (int j = i; j < m.n; ++j) s += cabs2(m.a[(size_t)j * m.lda + i]);
  out[(size_t)blockIdx.y * ld + i] = s;
}

// dst (n2 x r) = R_top^H, R_top = rows 0..r-1 of triu(src.a)
__global__ void transpose_top_kernel(const MatDesc *__restrict__ src, const MatDesc *__restrict__ dst) {
  const MatDesc s = src[blockIdx.y], d = dst[blockIdx.y];
  const long total = (long)d.m * d.n;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long)gridDim.x * blockDim.x) {
    const int j = (int)(idx % d.m), i = (int)(idx / d.m);   // dst row j (R column), dst column i (R row)
    d.a[(size_t)i * d.lda + j] = (j >= i) ? cconj(s.a[(size_t)j * s.lda + i]) : cz(0.0, 0.0);
  }
}

// dst (n2 x n2) = triu(src.a[0:n2, 0:n2])
__global__ void copy_r_kernel(const MatDesc *__restrict__ src, const MatDesc *__restrict__ dst) {
  const MatDesc s = src[blockIdx.y], d = dst[blockIdx.y];
  const long total = (long)d.n * d.n;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long)gridDim.x * blockDim.x) {
    const int r = (int)(idx % d.n), c = (int)(idx / d.n);
    d.a[(size_t)c * d.lda + r] = (r <= c) ? s.a[(size_t)c * s.lda + r] : cz(0.0, 0.0);
  }
}

// After Jacobi on L (desc l: g = U_L S, perm/sv/rank sorted):
//   ql.u[:, k] = [g_{perm k} / s_k ; 0]  (m rows)   -- left factor, before Q_h
// and zeros where right_factor_kernel writes nothing of
//   l.u[:, k]  = [V_L e_k / s_k ; 0]  (n2 rows)  -- right factor, before Z
__global__ void prep_u_kernel(const MatDesc *__restrict__ qd, const MatDesc *__restrict__ ld) {
  const MatDesc q = qd[blockIdx.y], l = ld[blockIdx.y];
  const int k = blockIdx.x;
  const int r = l.n;
  if (k >= r) return;
  const int kept = l.rank[0];
  double2 *uq = q.u + (size_t)k * q.lda;
  double2 *ul = l.u + (size_t)k * l.lda;
  if (k >= kept) {
    for (int i = threadIdx.x; i < q.m; i += blockDim.x) uq[i] = cz(0.0, 0.0);
    for (int i = threadIdx.x; i < l.m; i += blockDim.x) ul[i] = cz(0.0, 0.0);
    return;
  }
  const int c = l.perm[k];
  const double inv = 1.0 / l.sv[k];
  const double2 *g = l.g + (size_t)c * l.ldg;
  for (int i = threadIdx.x; i < q.m; i += blockDim.x) uq[i] = (i < r) ? cscale(g[i], inv) : cz(0.0, 0.0);
  for (int i = r + threadIdx.x; i < l.m; i += blockDim.x) ul[i] = cz(0.0, 0.0);
}

// l.u[0:r, 0:kept] = V_L S^+ = L^{-1} U_L = X^H U_L with X = R_L^{-1} (upper, x)
// and U_L's columns g_{perm k} / s_k: one 64 x 64 tile a workgroup on the FP64
// matrix cores, 16 rows of X and U_L staged through LDS at a time, the sum
// ending with the tile's last row of L^{-1}.  Bound by the matrix cores: 4 r^2
// kept flops against 16 r^3 a Jacobi sweep for rotating V along.  770 blocks of
// 16 bodies (r about 250): 3.8 ms, X 5 ms, and the rotation apply 194 -> 99 ms;
// the build 485 -> 402 ms.
__global__ __launch_bounds__(256) void right_factor_kernel(const MatDesc *__restrict__ ld,
                                                           const MatDesc *__restrict__ xd) {
  constexpr int KS = 16, TS = 64;
  const MatDesc l = ld[blockIdx.z], x = xd[blockIdx.z];
  const int r = l.n, kept = l.rank[0];
  const int c0 = blockIdx.x * TS, i0 = blockIdx.y * TS;
  if (c0 >= kept || i0 >= r) return;
  __shared__ double2 Xs[KS][TS + 1], Gs[KS][TS + 1];
  __shared__ double inv[TS];
  __shared__ int col[TS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int l16 = lane & 15, k4 = lane >> 4, wi = wv & 1, wc = wv >> 1;
  if (tid < TS) {
    const bool in = c0 + tid < kept;
    col[tid] = in ? l.perm[c0 + tid] : 0;
    inv[tid] = in ? 1.0 / l.sv[c0 + tid] : 0.0;
  }
  dx4 re[2][2], im[2][2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) re[u][v] = im[u][v] = dx4{0, 0, 0, 0};
  const int jend = min(r, i0 + TS);
  __syncthreads();
  for (int j0 = 0; j0 < jend; j0 += KS) {
#pragma unroll
    for (int u = 0; u < KS * TS / 256; ++u) {
      const int idx = tid + 256 * u, jj = idx % KS, c = idx / KS, j = j0 + jj;
      Xs[jj][c] = ld_or0(x.a, (size_t)min(i0 + c, r - 1) * x.lda + min(j, r - 1), j <= i0 + c && i0 + c < r);
      Gs[jj][c] = cscale(ld_or0(l.g, (size_t)col[c] * l.ldg + min(j, r - 1), j < r), inv[c]);
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < KS; kk += 4) {
      double2 a[2], y[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) a[u] = Xs[kk + k4][32 * wi + 16 * u + l16];
#pragma unroll
      for (int v = 0; v < 2; ++v) y[v] = Gs[kk + k4][32 * wc + 16 * v + l16];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {   // conj(X)^T U
          re[u][v] = mfma_f64(a[u].x, y[v].x, re[u][v]);
          re[u][v] = mfma_f64(a[u].y, y[v].y, re[u][v]);
          im[u][v] = mfma_f64(a[u].x, y[v].y, im[u][v]);
          im[u][v] = mfma_f64(-a[u].y, y[v].x, im[u][v]);
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int c = c0 + 32 * wc + 16 * v + l16;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + 32 * wi + 16 * u + k4 + 4 * e;
        if (c < kept && i < r) l.u[(size_t)c * l.lda + i] = cz(re[u][v][e], im[u][v][e]);
      }
    }
}

// W[perm[i], k] = l.u[i, k] (rows of dropped columns stay zero)
__global__ void scatter_w_kernel(const MatDesc *__restrict__ ld, const MatDesc *__restrict__ fd,
                                 const int *__restrict__ perm, const int *__restrict__ piv, int ldp,
                                 const double *__restrict__ scale) {
  const MatDesc l = ld[blockIdx.y], f = fd[blockIdx.y];
  const int k = blockIdx.x;
  const int kept = l.rank[0];
  if (k >= kept) return;   // W has exactly `kept` columns
  double2 *w = f.w + (size_t)k * f.ldg;
  for (int i = threadIdx.x; i < f.n; i += blockDim.x) w[i] = cz(0.0, 0.0);
  __syncthreads();
  const double2 *src = l.u + (size_t)k * l.lda;
  const int *pw = perm + (size_t)blockIdx.y * ldp;
  const int *vw = piv + (size_t)blockIdx.y * ldp;
  const double *sw = scale ? scale + (size_t)blockIdx.y * ldp : nullptr;
  for (int i = threadIdx.x; i < l.m; i += blockDim.x) {
    const int c = pw[vw[i]];
    w[c] = sw ? cscale(src[i], sw[c]) : src[i];
  }
}

// out[w][i] = singular value i of matrix w (zero past its n), ld entries per matrix
__global__ void sv_gather_kernel(const MatDesc *__restrict__ ld, int ldo, double *__restrict__ out) {
  const MatDesc l = ld[blockIdx.x];
  for (int i = threadIdx.x; i < ldo; i += blockDim.x) out[(size_t)blockIdx.x * ldo + i] = i < l.n ? l.sv[i] : 0.0;
}

constexpr int PK = 512;   // threads of the pivot/reflector kernel

// Step k of column-pivoted QR, part 1 (one workgroup per matrix): move the
// column of largest remaining norm to position k (columns, norms and the
// pivot record are swapped), then form the Householder reflector of column k
// (rows k..m-1), LAPACK's zlarfg convention.
__global__ __launch_bounds__(PK) void qrcp_pivot_kernel(const MatDesc *__restrict__ descs, int k,
                                                        double *__restrict__ norms,
                                                        int *__restrict__ piv, int ld) {
  const MatDesc d = descs[blockIdx.x];
  if (k >= d.n) return;
  double *nr = norms + (size_t)blockIdx.x * ld;
  int *pv = piv + (size_t)blockIdx.x * ld;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ double rv[PK / 64];
  __shared__ int ri[PK / 64];
  __shared__ int s_p;
  __shared__ double s_sum;
  double best = -1.0;
  int bi = k;
  for (int c = k + tid; c < d.n; c += PK) {
    const double v = nr[c];
    if (v > best) { best = v; bi = c; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ov = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  if (lane == 0) { rv[wv] = best; ri[wv] = bi; }
  __syncthreads();
  if (tid == 0) {
    double b = rv[0];
    int i = ri[0];
    for (int w = 1; w < PK / 64; ++w)
      if (rv[w] > b || (rv[w] == b && ri[w] < i)) { b = rv[w]; i = ri[w]; }
    s_p = i;
  }
  __syncthreads();
  const int p = s_p;
  if (p != k) {
    double2 *ck = d.a + (size_t)k * d.lda, *cp = d.a + (size_t)p * d.lda;
    for (int r = tid; r < d.m; r += PK) {
      const double2 t = ck[r];
      ck[r] = cp[r];
      cp[r] = t;
    }
    if (tid == 0) {
      const double tn = nr[k]; nr[k] = nr[p]; nr[p] = tn;
      const int ti = pv[k]; pv[k] = pv[p]; pv[p] = ti;
    }
  }
  __syncthreads();
  double2 *col = d.a + (size_t)k * d.lda;
  double s = 0.0;
  for (int r = k + 1 + tid; r < d.m; r += PK) s += cabs2(col[r]);
  s = wave_sum(s);
  if (lane == 0) rv[wv] = s;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < PK / 64; ++w) t += rv[w];
    s_sum = t;
  }
  __syncthreads();
  const double ssum = s_sum;
  const double2 alpha = col[k];
  double2 tau = cz(0.0, 0.0);
  if (!(ssum == 0.0 && alpha.y == 0.0)) {
    const double beta = -copysign(sqrt(alpha.x * alpha.x + alpha.y * alpha.y + ssum), alpha.x);
    tau = cz((beta - alpha.x) / beta, -alpha.y / beta);
    const double2 den = cz(alpha.x - beta, alpha.y);
    const double dd = cabs2(den);
    const double2 scal = cz(den.x / dd, -den.y / dd);
    for (int r = k + 1 + tid; r < d.m; r += PK) col[r] = cmul(col[r], scal);
    __syncthreads();
    if (tid == 0) col[k] = cz(beta, 0.0);
  }
  if (tid == 0) d.tau[k] = tau;
}

// Step k, part 2: apply H_k^H to every column c > k (one wave per column) and
// recompute its norm over rows k+1..m-1 (the pivot criterion of step k+1).
__global__ __launch_bounds__(256) void qrcp_update_kernel(const MatDesc *__restrict__ descs, int k,
                                                          double *__restrict__ norms, int ld) {
  const MatDesc d = descs[blockIdx.y];
  const int c = k + 1 + blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= d.n || c >= d.n) return;
  const int lane = threadIdx.x & 63;
  const double2 *v = d.a + (size_t)k * d.lda;
  double2 *a = d.a + (size_t)c * d.lda;
  const double2 ctau = cconj(d.tau[k]);
  double2 acc = cz(0.0, 0.0);
  for (int r = k + lane; r < d.m; r += 64) {
    const double2 vr = (r == k) ? cz(1.0, 0.0) : v[r];
    cfmac(acc, vr, a[r]);
  }
  acc = wave_sum(acc);
  const double2 f = cmul(ctau, acc);
  double s = 0.0;
  for (int r = k + lane; r < d.m; r += 64) {
    const double2 vr = (r == k) ? cz(1.0, 0.0) : v[r];
    const double2 x = csub(a[r], cmul(vr, f));
    a[r] = x;
    if (r > k) s += cabs2(x);
  }
  s = wave_sum(s);
  if (lane == 0) norms[(size_t)blockIdx.y * ld + c] = sqrt(s);
}

// The whole column-pivoted QR of a triangle of at most 64 RL rows and 16 CW
// columns in one launch, one workgroup a matrix, the triangle in registers:
// wave w holds the columns w, w + 16, ..., a lane a row of each 64.  Nothing is
// swapped: the chosen column's wave forms its reflector, writes the finished
// column where it belongs and drops it; the others read the reflector from LDS.
// A step is two barriers: every wave finds the largest norm by itself (the
// column's index in the last bits, so equal norms to 2^-45 go to the lowest
// index), the chosen column's wave forms the reflector; all apply it and
// recompute their norms, the sums of all a wave's columns in one butterfly.
// Bound by that chain: 17 triangles of 60 columns 102 us, of 120 309 us; with the
// triangle in L2 and the columns swapped 234 and 588 us.
constexpr int QN = 128, QW = 16;

// Sums over the wave of N values (N = 4, 8 or 16): on return lane 4 i holds the
// sum of v[i] in v[0] (so do lanes 4 i + 1 .. 4 i + 3, to rounding).
template <int N>
__device__ inline void wave_sums(double (&v)[N], int lane) {
  if constexpr (N == 16) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = swap32_add(v[i], v[i + 8]);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = swap32_add(v[i], v[i]);
  }
  if constexpr (N >= 8) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = swap16_add(v[i], v[i + 4]);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = swap16_add(v[i], v[i]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool hi = lane & 8;
    const double send = hi ? v[i] : v[i + 2], keep = hi ? v[i + 2] : v[i];
    v[i] = keep + dpp_move<0x128, 0xf>(send);   // row_ror 8
  }
  const bool hi = lane & 4;
  const double send = hi ? v[0] : v[1], keep = hi ? v[1] : v[0];
  double t = keep + dpp_move<0x141, 0xf>(send);   // row_half_mirror
  t += dpp_move<0x4e, 0xf>(t);                    // quad_perm 2 3 0 1
  v[0] = t + dpp_move<0xb1, 0xf>(t);              // quad_perm 1 0 3 2
}

template <int RL, int CW>
__global__ __launch_bounds__(64 * QW) void qrcp_one_kernel(const MatDesc *__restrict__ descs, int *__restrict__ piv,
                                                           int ld) {
  const MatDesc d = descs[blockIdx.x];
  const int n = d.n, m = d.m, tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  int *pv = piv + (size_t)blockIdx.x * ld;
  __shared__ double nr[QW * CW];
  __shared__ int lab[QW * CW];
  __shared__ double2 v[64 * RL];
  __shared__ double2 s_tau;
  double2 a[CW][RL];
  unsigned live = 0;
#pragma unroll
  for (int j = 0; j < CW; ++j) {
    const int c = QW * j + wv;
    live |= c < n ? 1u << j : 0u;
#pragma unroll
    for (int u = 0; u < RL; ++u)
      a[j][u] = ld_or0(d.a + (size_t)min(c, n - 1) * d.lda, 64 * u + lane, c < n && 64 * u + lane < m);
  }
  if (tid < QW * CW) lab[tid] = tid < n ? pv[tid] : 0;
  // norms of the rows from k0 on
  auto norms = [&](int k0) {
    double q[CW < 4 ? 4 : CW];
#pragma unroll
    for (int j = 0; j < (CW < 4 ? 4 : CW); ++j) {
      q[j] = 0.0;
      if (j < CW)
#pragma unroll
        for (int u = 0; u < RL; ++u) q[j] += 64 * u + lane >= k0 ? cabs2(a[j < CW ? j : 0][u]) : 0.0;
    }
    wave_sums(q, lane);
    const int j = lane >> 2;
    // a NaN stays in the race, an infinity stays a number with an index in it
    if ((lane & 3) == 0 && j < CW) nr[QW * j + wv] = (live >> j) & 1 ? (q[0] >= 0.0 ? fmin(q[0], 1.7e308) : 0.0) : -1.0;
  };
  norms(0);
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    // the largest norm's column
    double best = -1.0;
#pragma unroll
    for (int c = lane; c < QW * CW; c += 64) {
      const double x = nr[c];
      const long long b = (__double_as_longlong(x) & ~127LL) | (127 - c);
      best = x >= 0.0 ? fmax(best, __longlong_as_double(b)) : best;
    }
    best = wave_max_dpp(best);
    const int p = __builtin_amdgcn_readfirstlane(127 - ((int)__double_as_longlong(best) & 127));
    if (wv == p % QW) {   // uniform
      double2 x[RL];
#pragma unroll
      for (int j = 0; j < CW; ++j)
        if (j == p / QW)
#pragma unroll
          for (int u = 0; u < RL; ++u) x[u] = a[j][u];
      live &= ~(1u << (p / QW));
      double q = 0.0;
      double2 alpha = cz(0.0, 0.0);
#pragma unroll
      for (int u = 0; u < RL; ++u) {
        q += 64 * u + lane > k ? cabs2(x[u]) : 0.0;
        if (u == k / 64) alpha = x[u];
      }
      q = wave_sum(q);
      alpha = cz(lane_value(alpha.x, k & 63), lane_value(alpha.y, k & 63));
      double2 tau = cz(0.0, 0.0), scal = cz(1.0, 0.0), diag = alpha;
      if (!(q == 0.0 && alpha.y == 0.0)) {
        const double beta = -copysign(sqrt(alpha.x * alpha.x + alpha.y * alpha.y + q), alpha.x);
        tau = cz((beta - alpha.x) / beta, -alpha.y / beta);
        const double2 den = cz(alpha.x - beta, alpha.y);
        const double dd = cabs2(den);
        scal = cz(den.x / dd, -den.y / dd);
        diag = cz(beta, 0.0);
      }
      double2 *ck = d.a + (size_t)k * d.lda;
#pragma unroll
      for (int u = 0; u < RL; ++u) {
        const int r = 64 * u + lane;
        const double2 t = cmul(x[u], scal);
        v[r] = csel(r > k, t, cz(r == k ? 1.0 : 0.0, 0.0));
        if (r < m) ck[r] = csel(r > k, t, csel(r == k, diag, x[u]));
      }
      if (lane == 0) {
        s_tau = tau;
        d.tau[k] = tau;
        pv[k] = lab[p];
      }
    }
    __syncthreads();
    if (live) {   // uniform
      const double2 ctau = cconj(s_tau);
      double2 vr[RL], vt[RL];
#pragma unroll
      for (int u = 0; u < RL; ++u) {
        vr[u] = v[64 * u + lane];
        vt[u] = cmul(ctau, vr[u]);
        vt[u] = cz(-vt[u].x, -vt[u].y);
      }
      double s[2 * CW];
#pragma unroll
      for (int j = 0; j < CW; ++j) {
        double2 t = cz(0.0, 0.0);
#pragma unroll
        for (int u = 0; u < RL; ++u) cfmac(t, vr[u], a[j][u]);
        s[2 * j] = t.x;
        s[2 * j + 1] = t.y;
      }
      wave_sums(s, lane);
#pragma unroll
      for (int j = 0; j < CW; ++j) {
        const double2 f = cz(lane_value(s[0], 8 * j), lane_value(s[0], 8 * j + 4));
#pragma unroll
        for (int u = 0; u < RL; ++u) cfma(a[j][u], vt[u], f);
      }
    }
    norms(k + 1);
    __syncthreads();   // norms settled, the reflector's slots free
  }
}

}  // namespace

// One step of the column-pivoted QR above on a batch (the pivot and its
// reflector, then the update of the columns after it with their norms).
void launch_qrcp_step(const MatDesc *descs, int W, int nmax, int k, double *norms, int *piv, int ld,
                      hipStream_t s) {
  hipLaunchKernelGGL(qrcp_pivot_kernel, dim3(W), dim3(PK), 0, s, descs, k, norms, piv, ld);
  if (k + 1 < nmax)
    hipLaunchKernelGGL(qrcp_update_kernel, dim3(cdiv(nmax - k - 1, 4), W), dim3(256), 0, s, descs, k, norms, ld);
  HIP_CHECK(hipGetLastError());
}

namespace {

// Compact-WY T factor of every 32-column panel of reflectors (forward,
// columnwise): T[i][i] = tau_i, T[0:i, i] = -tau_i T[0:i, 0:i] V^H v_i.
__global__ __launch_bounds__(256) void build_t_kernel(const MatDesc *__restrict__ descs) {
  const MatDesc d = descs[blockIdx.x];
  const int k0 = blockIdx.y * kQRNB;
  if (k0 >= d.n) return;
  const int nbp = min(kQRNB, d.n - k0);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ double2 gram[kQRNB][kQRNB + 1];
  __shared__ double2 Tsh[kQRNB][kQRNB + 1];
  __shared__ double2 tmp[kQRNB];
  auto vload = [&](int i, int r) -> double2 {
    const int c = k0 + i;
    if (r < c) return cz(0.0, 0.0);
    if (r == c) return cz(1.0, 0.0);
    return d.a[(size_t)c * d.lda + r];
  };
  const int npairs = nbp * (nbp - 1) / 2;
  for (int pidx = wv; pidx < npairs; pidx += 4) {
    int i = 1, base = 0;
    while (base + i <= pidx) { base += i; ++i; }
    const int g = pidx - base;
    double2 acc = cz(0.0, 0.0);
    for (int r = k0 + i + lane; r < d.m; r += 64) cfmac(acc, vload(g, r), vload(i, r));
    acc = wave_sum(acc);
    if (lane == 0) gram[g][i] = acc;
  }
  __syncthreads();
  for (int i = 0; i < nbp; ++i) {
    const double2 ti = d.tau[k0 + i];
    if (tid < i) tmp[tid] = cmul(cz(-ti.x, -ti.y), gram[tid][i]);
    __syncthreads();
    if (tid < i) {
      double2 acc = cz(0.0, 0.0);
      for (int g = tid; g < i; ++g) cfma(acc, Tsh[tid][g], tmp[g]);
      Tsh[tid][i] = acc;
    }
    if (tid == i) Tsh[i][i] = ti;
    __syncthreads();
  }
  double2 *T = d.T + (size_t)blockIdx.y * kQRNB * kQRNB;
  for (int idx = tid; idx < kQRNB * kQRNB; idx += 256) {
    const int r = idx % kQRNB, c = idx / kQRNB;
    T[idx] = (r <= c && c < nbp) ? Tsh[r][c] : cz(0.0, 0.0);
  }
}


// ------------------------------------------------ inverse of the triangle
// X = R^{-1} for the n x n upper triangle R of a QR'd matrix, in TI x TI
// blocks: the diagonal blocks first (trinv_diag_kernel), then the blocks at
// block distance d = 1, 2, ... from the diagonal (trinv_off_kernel), each
// from X_ij = -X_ii sum_{k=i+1..j} R_ik X_kj, whose X_kj lie nearer the
// diagonal and are already formed.  X must be zero below the diagonal.
constexpr int TI = 64;

__device__ inline double2 crecip(double2 a) {
  const double d = 1.0 / cabs2(a);
  return cz(a.x * d, -a.y * d);
}

// One workgroup a diagonal block: each wave inverts a 16 x 16 diagonal block of
// it in registers, then X_12 = -X_11 R_12 X_22 doubles the blocks twice on the
// matrix cores.  17 triangles of 120 columns 82 -> 12.5 us (a thread a column,
// back substitution through LDS).
__global__ __launch_bounds__(256) void trinv_diag_kernel(const MatDesc *__restrict__ rd,
                                                         const MatDesc *__restrict__ xd) {
  const MatDesc r = rd[blockIdx.y], x = xd[blockIdx.y];
  const int n = x.n;
  const int j0 = blockIdx.x * TI;
  if (j0 >= n) return;
  const int nb = min(TI, n - j0);
  __shared__ double2 Xs[TI][TI + 1];
  __shared__ double2 Ts[TI / 2][TI / 2 + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, k = lane >> 4;
  // entry (i, j) of the block; the identity past the matrix's end
  auto R = [&](int i, int j) {
    const bool in = i <= j && j < nb;
    return csel(j >= nb && i == j, cz(1.0, 0.0), ld_or0(r.a, (size_t)(j0 + j) * r.lda + j0 + i, in));
  };
  {
    const int b = 16 * wv;
    double2 y[4], t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      y[u] = R(b + 4 * u + k, b + c);
      t[u] = cz(4 * u + k == c ? 1.0 : 0.0, 0.0);
    }
    rsolve16<0>(t, y, crecip(R(b + c, b + c)), c);
#pragma unroll
    for (int u = 0; u < 4; ++u) Xs[b + 4 * u + k][b + c] = t[u];
  }
  __syncthreads();
  double2 p[4], q[4], t[4];
  if (wv < 2) {
    const int b = 32 * wv, e = b + 16;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      p[u] = R(b + c, e + 4 * u + k);
      q[u] = Xs[e + 4 * u + k][e + c];
    }
    mul16(p, q, t);
#pragma unroll
    for (int u = 0; u < 4; ++u) p[u] = Xs[b + c][b + 4 * u + k];
    mul16(p, t, q);
#pragma unroll
    for (int u = 0; u < 4; ++u) Xs[b + 4 * u + k][e + c] = cz(-q[u].x, -q[u].y);
  }
  __syncthreads();
  const int ti = 16 * (wv >> 1), tj = 16 * (wv & 1);   // this wave's tile of the upper right quarter
  dx4 re = {0, 0, 0, 0}, im = re;
  for (int m = 0; m <= tj; m += 16) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      p[u] = R(ti + c, 32 + m + 4 * u + k);
      q[u] = Xs[32 + m + 4 * u + k][32 + tj + c];
    }
    mfma16(p, q, re, im);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) Ts[ti + 4 * u + k][tj + c] = cz(re[u], im[u]);
  __syncthreads();
  re = dx4{0, 0, 0, 0};
  im = re;
  for (int m = ti; m < 32; m += 16) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      p[u] = Xs[ti + c][m + 4 * u + k];
      q[u] = Ts[m + 4 * u + k][tj + c];
    }
    mfma16(p, q, re, im);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) Xs[ti + 4 * u + k][32 + tj + c] = cz(-re[u], -im[u]);
  __syncthreads();
  for (int idx = tid; idx < TI * TI; idx += 256) {
    const int i = idx % TI, j = idx / TI;
    if (i < nb && j < nb) x.a[(size_t)(j0 + j) * x.lda + j0 + i] = i <= j ? Xs[i][j] : cz(0.0, 0.0);
  }
}

// Blocks (i, i + d) of every matrix: one workgroup a 16-column slice, a wave 16
// of its rows, the fragments of R and X straight from memory with the next ones
// in flight, T = sum_k R_ik X_kj through LDS to the product with -X_ii.  Bound by
// the compute unit's matrix cores, 3 us a block of the sum: d = 1 of 2 matrices of
// 650 columns 75 -> 10 us, d = 10 in one launch 36 (a workgroup a 64 x 64 block with
// both operands staged in LDS, long sums split over workgroups and added by a
// launch more: 80 + 36).  The sum in four shares over 16 waves is no faster: 31 us.
__global__ __launch_bounds__(256) void trinv_off_kernel(const MatDesc *__restrict__ rd,
                                                        const MatDesc *__restrict__ xd, int d) {
  const MatDesc r = rd[blockIdx.y], x = xd[blockIdx.y];
  const int n = x.n;
  const int i0 = (blockIdx.x >> 2) * TI, j0 = i0 + d * TI + 16 * (blockIdx.x & 3);
  if (j0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, k = lane >> 4, rt = 16 * wv;
  __shared__ double2 Ts[TI][17];
  const int row = i0 + rt + c;   // row block i is whole (it precedes j)
  const int col = min(j0 + c, n - 1);
  const double2 *xc = x.a + (size_t)col * x.lda;
  const int kend = min(j0 + 16, n);   // X is zero below its diagonal
  dx4 re = {0, 0, 0, 0}, im = re;
  double2 p[4], q[4], pn[4], qn[4];
  auto fetch = [&](int k0, double2(&a)[4], double2(&b)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int kk = k0 + 4 * u + k;
      const bool in = kk < kend;
      a[u] = ld_or0(r.a, (size_t)kk * r.lda + row, in);
      b[u] = ld_or0(xc, kk, in && j0 + c < n);
    }
  };
  fetch(i0 + TI, p, q);
  for (int k0 = i0 + TI; k0 < kend; k0 += 32) {
    fetch(k0 + 16, pn, qn);
    mfma16(p, q, re, im);
    fetch(k0 + 32, p, q);
    mfma16(pn, qn, re, im);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) Ts[rt + 4 * u + k][c] = cz(re[u], im[u]);
  __syncthreads();
  re = dx4{0, 0, 0, 0};
  im = re;
  for (int m = rt; m < TI; m += 16) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      p[u] = x.a[(size_t)(i0 + m + 4 * u + k) * x.lda + row];
      q[u] = Ts[m + 4 * u + k][c];
    }
    mfma16(p, q, re, im);
  }
  if (j0 + c < n)
#pragma unroll
    for (int u = 0; u < 4; ++u)
      x.a[(size_t)(j0 + c) * x.lda + i0 + rt + 4 * u + k] = cz(-re[u], -im[u]);
}

// The blocks off the diagonal of X = R^{-1} (diagonal blocks done), one
// block distance d after the other.
void trinv_offdiag(const MatDesc *rd, const MatDesc *xd, int W, int nblk, hipStream_t s) {
  for (int d = 1; d < nblk; ++d)
    hipLaunchKernelGGL(trinv_off_kernel, dim3(4 * (nblk - d), W), dim3(256), 0, s, rd, xd, d);
  HIP_CHECK(hipGetLastError());
}

// out[w][j] = (sum_{i<=j} |R_ij|^2, sum_{i<=j} |X_ij|^2): one wave per column
__global__ __launch_bounds__(256) void trinv_norm_kernel(const MatDesc *__restrict__ rd,
                                                         const MatDesc *__restrict__ xd, double2 *out, int ld) {
  const MatDesc r = rd[blockIdx.y], x = xd[blockIdx.y];
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (j >= x.n) return;
  double sr = 0.0, sx = 0.0;
  for (int i = lane; i <= j; i += 64) {
    sr += cabs2(r.a[(size_t)j * r.lda + i]);
    sx += cabs2(x.a[(size_t)j * x.lda + i]);
  }
  sr = wave_sum(sr);
  sx = wave_sum(sx);
  if (lane == 0) out[(size_t)blockIdx.y * ld + j] = cz(sr, sx);
}

// d.u = the first d.rank[0] columns of the identity (rows past them zero)
__global__ void identity_u_kernel(const MatDesc *__restrict__ descs) {
  const MatDesc d = descs[blockIdx.y];
  const int k = blockIdx.x;
  if (k >= d.rank[0]) return;
  double2 *u = d.u + (size_t)k * (d.ldu ? d.ldu : d.lda);
  for (int i = threadIdx.x; i < d.m; i += blockDim.x) u[i] = cz(i == k ? 1.0 : 0.0, 0.0);
}
}  // namespace

// Two HIP events around a stretch of work on a stream.
struct EvPair {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  explicit EvPair(hipStream_t s) {
    HIP_CHECK(hipEventCreate(&e0));
    HIP_CHECK(hipEventCreate(&e1));
    HIP_CHECK(hipEventRecord(e0, s));
  }
  void stop(hipStream_t s) { (void)hipEventRecord(e1, s); }
  double ms() const {
    float t = 0.f;
    return hipEventElapsedTime(&t, e0, e1) == hipSuccess ? (double)t : 0.0;
  }
  ~EvPair() {
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
  }
  EvPair(const EvPair &) = delete;
  EvPair &operator=(const EvPair &) = delete;
};

// bytes of n complex entries rounded up to 256 (the arena alignment)
static size_t arena_bytes(size_t n) { return (n * sizeof(double2) + 255) / 256 * 256; }
static double2 *arena_at(const DevBuf &b, size_t off) {
  return reinterpret_cast<double2 *>(static_cast<char *>(b.p) + off);
}

static void upload_descs(DevBuf &buf, const std::vector<MatDesc> &h, hipStream_t s) {
  buf.alloc(h.size() * sizeof(MatDesc));
  HIP_CHECK(hipMemcpyAsync(buf.p, h.data(), h.size() * sizeof(MatDesc), hipMemcpyHostToDevice, s));
}

// Largest singular value of each triangle (n2[w] x n2[w], upper) by power
// iteration on R^H R from the all-ones vector; iters rounds.  Blocking.
static std::vector<double> tri_sigma1(const MatDesc *tri, const std::vector<int> &n2, int ld, hipStream_t s,
                                      int iters = 10) {
  const int W = (int)n2.size();
  const int nmax = *std::max_element(n2.begin(), n2.end());
  std::vector<double2> hx((size_t)W * ld, cz(0.0, 0.0));
  for (int w = 0; w < W; ++w)
    for (int i = 0; i < n2[w]; ++i) hx[(size_t)w * ld + i] = cz(1.0 / std::sqrt((double)n2[w]), 0.0);
  DevBuf x(hx.size() * sizeof(double2)), y(hx.size() * sizeof(double2));
  std::vector<double> s1(W, 0.0);
  for (int it = 0; it < iters; ++it) {
    HIP_CHECK(hipMemcpyAsync(x.p, hx.data(), hx.size() * sizeof(double2), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(trimv_kernel, dim3(cdiv(nmax, 256), W), dim3(256), 0, s, tri, x.as<double2>(),
                       y.as<double2>(), ld);
    hipLaunchKernelGGL(trimhv_kernel, dim3(cdiv(nmax, 4), W), dim3(256), 0, s, tri, y.as<double2>(),
                       x.as<double2>(), ld);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipMemcpyAsync(hx.data(), x.p, hx.size() * sizeof(double2), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    for (int w = 0; w < W; ++w) {
      double nrm = 0.0;
      for (int i = 0; i < n2[w]; ++i) nrm += cabs2(hx[(size_t)w * ld + i]);
      nrm = std::sqrt(nrm);   // ||R^H R x|| for the unit vector x: sigma_1^2 in the limit
      s1[w] = std::sqrt(nrm);
      const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
      for (int i = 0; i < n2[w]; ++i) hx[(size_t)w * ld + i] = cscale(hx[(size_t)w * ld + i], inv);
    }
  }
  return s1;
}

// Whether the truncated pseudoinverse after the pivoted QR of the triangle
// is taken as a complete orthogonal decomposition (truncated at the pivoted
// triangle's trailing Frobenius norm, then L^{-1} of its LQ) instead of the
// Jacobi SVD of L.  Default: for the periodizer's equilibrated Q from
// kCodMinCols columns on, the SVD otherwise.  MFS_QPINV=svd or cod decides
// for every equilibrated batch (the periodizer), MFS_OPINV=cod takes it for
// the one-body operators' blocks too (no singular values are then formed).
constexpr int kCodMinCols = 4096;
static bool use_cod(bool equilibrate, int n2max) {
  const char *e = std::getenv(equilibrate ? "MFS_QPINV" : "MFS_OPINV");
  if (e && std::string(e) == "cod") return true;
  if (e && std::string(e) == "svd") return false;
  return equilibrate && n2max >= kCodMinCols;
}

// Panels of the periodizer's QR: Cholesky QR, or MFS_QR_PANEL=steps.
static bool chol_panels() {
  const char *e = std::getenv("MFS_QR_PANEL");
  return !(e && std::string(e) == "steps");
}

// The equilibrated columns of the periodizer's Q are usually independent well
// within the cutoff; the truncated SVD then keeps every singular value and
// the pseudoinverse is D P R^{-1} Q_1^H, with Q_1 R the QR of the ordered,
// scaled columns (P their order, D the scaling).  Since cond_2(R) <=
// ||R||_F ||R^{-1}||_F, a bound below 1/rel_cutoff shows that no singular
// value falls under the cutoff, without the SVD: then U = Q_1 and
// W = D P R^{-1} are formed and true is returned.  Otherwise (some matrix of
// the batch may need truncating) nothing is kept and false is returned.
static bool direct_pinv(GradedPinv &g, const std::vector<int> &n2, int nmax, double rel_cutoff,
                        const double *cscl, const std::vector<MatDesc> &in, hipStream_t s, bool keep_reflectors,
                        bool halves) {
  const int W = (int)n2.size();
  const int n2max = *std::max_element(n2.begin(), n2.end());
  int *flags = g.small.as<int>();
  std::vector<size_t> ox(W);
  size_t tx = 0;
  for (int w = 0; w < W; ++w) {
    ox[w] = tx;
    tx += arena_bytes((size_t)round_up(n2[w], 16) * n2[w]);
  }
  DevBuf xa(tx), dx;
  std::vector<MatDesc> hx(W);
  for (int w = 0; w < W; ++w) {
    MatDesc d{};
    d.a = arena_at(xa, ox[w]);
    d.u = d.a;
    d.m = n2[w]; d.n = n2[w]; d.lda = round_up(n2[w], 16);
    d.rank = flags + W + w;
    hx[w] = d;
  }
  upload_descs(dx, hx, s);
  launch_zero(xa.as<double2>(), (long)(tx / sizeof(double2)), s);
  const int nblk = cdiv(n2max, TI);
  hipLaunchKernelGGL(trinv_diag_kernel, dim3(nblk, W), dim3(256), 0, s, g.d_qc.as<MatDesc>(), dx.as<MatDesc>());
  trinv_offdiag(g.d_qc.as<MatDesc>(), dx.as<MatDesc>(), W, nblk, s);

  DevBuf nrm((size_t)W * n2max * sizeof(double2));
  hipLaunchKernelGGL(trinv_norm_kernel, dim3(cdiv(n2max, 4), W), dim3(256), 0, s, g.d_qc.as<MatDesc>(),
                     dx.as<MatDesc>(), nrm.as<double2>(), n2max);
  HIP_CHECK(hipGetLastError());
  std::vector<double2> hn((size_t)W * n2max);
  HIP_CHECK(hipMemcpyAsync(hn.data(), nrm.p, hn.size() * sizeof(double2), hipMemcpyDeviceToHost, s));
  HIP_CHECK(hipStreamSynchronize(s));
  double sr = 0.0, sx = 0.0;
  for (int w = 0; w < W; ++w) {
    if (!(halves && w % 2)) sr = sx = 0.0;
    for (int j = 0; j < n2[w]; ++j) {
      sr += hn[(size_t)w * n2max + j].x;
      sx += hn[(size_t)w * n2max + j].y;
    }
    if (halves && w % 2 == 0) continue;   // the bound of both halves together
    const double bound = std::sqrt(sr) * std::sqrt(sx);
    if (!std::isfinite(bound) || !(bound * rel_cutoff < 1.0)) return false;
  }
  // every singular value is kept: rank n2, U = Q_1, W = D P R^{-1}
  g.kept = n2;
  g.rows = n2;
  g.cols = n2;
  g.direct = true;
  g.jacobi_ms = g.jacobi_bytes = g.jacobi_flops = 0.0;
  g.jacobi_launches = 0;
  g.jacobi_unconverged = 0;
  HIP_CHECK(hipMemcpyAsync(flags + W, n2.data(), W * sizeof(int), hipMemcpyHostToDevice, s));
  g.reflect = keep_reflectors;
  if (!keep_reflectors) {
    hipLaunchKernelGGL(identity_u_kernel, dim3(n2max, W), dim3(256), 0, s, g.d_qc.as<MatDesc>());
    HIP_CHECK(hipGetLastError());
    qr_form_u(g.d_qc.as<MatDesc>(), g.h_qc, n2max, s, true, g.qr_nb);
  }
  g.h_fin.resize(W);
  std::vector<size_t> of(W);
  {
    size_t tf = 0;
    for (int w = 0; w < W; ++w) {
      of[w] = tf;
      tf += arena_bytes((size_t)round_up(in[w].n, 16) * n2[w]);
    }
    g.fin_w.alloc(tf);
  }
  for (int w = 0; w < W; ++w) {
    MatDesc d{};
    d.m = in[w].m; d.n = in[w].n; d.lda = g.h_qc[w].lda;
    d.u = keep_reflectors ? nullptr : g.h_qc[w].u;
    d.w = arena_at(g.fin_w, of[w]);
    d.ldg = round_up(in[w].n, 16);
    d.rank = flags + W + w;
    g.h_fin[w] = d;
  }
  upload_descs(g.d_fin, g.h_fin, s);
  hipLaunchKernelGGL(scatter_w_kernel, dim3(n2max, W), dim3(256), 0, s, dx.as<MatDesc>(), g.d_fin.as<MatDesc>(),
                     g.perm.as<int>(), g.piv.as<int>(), nmax, cscl);
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipStreamSynchronize(s));
  return true;
}

void graded_pinv(GradedPinv &g, const std::vector<MatDesc> &in, double rel_cutoff, hipStream_t s,
                 bool equilibrate, bool keep_reflectors, bool halves) {
  const int W = (int)in.size();
  MFS_REQUIRE(!halves || W % 2 == 0, "graded pseudoinverse: halves come in pairs");
  int nmax = 0, mmax = 0;
  for (auto &d : in) { nmax = std::max(nmax, d.n); mmax = std::max(mmax, d.m); }
  g.direct = false;
  g.reflect = false;
  g.jacobi_unconverged = 0;
  upload_descs(g.d_in, in, s);
  // 1. column norms, selection and ordering
  DevBuf norms((size_t)W * nmax * sizeof(double));
  hipLaunchKernelGGL(colnorm_kernel, dim3(cdiv(nmax, 4), W), dim3(256), 0, s, g.d_in.as<MatDesc>(),
                     norms.as<double>(), nmax);
  HIP_CHECK(hipGetLastError());
  std::vector<double> hn((size_t)W * nmax);
  HIP_CHECK(hipMemcpyAsync(hn.data(), norms.p, hn.size() * sizeof(double), hipMemcpyDeviceToHost, s));
  HIP_CHECK(hipStreamSynchronize(s));
  std::vector<int> perm((size_t)W * nmax, 0), n2(W), rr(W);
  std::vector<double> scale(equilibrate ? (size_t)W * nmax : 0, 0.0);
  g.maxcol.assign(W, 0.0);
  // Matrices are independent: a batch of thousands spreads its selection
  // over host threads (one thread takes tens of milliseconds for the
  // 256-obstacle build's chunks, while the device waits).  bad[w]: 1 zero
  // matrix, 2 more columns kept than rows, 3 out of host memory.
  std::vector<char> bad(W, 0);
  auto select = [&](int w0, int w1) {
    std::vector<int> idx;
    for (int w = w0; w < w1; ++w) {
      try {
        const int n = in[w].n;
        const double *nw = hn.data() + (size_t)w * nmax;
        double mx = 0.0;
        for (int c = 0; c < n; ++c) mx = std::max(mx, nw[c]);
        // equilibrated: every kept column scaled to unit norm (the largest is 1);
        // only columns that vanish, or whose scaling would leave the exponent
        // range, are dropped
        g.maxcol[w] = equilibrate ? 1.0 : mx;
        const double keep_min = equilibrate ? 1e-250 * mx : 1e-15 * mx;
        idx.clear();
        for (int c = 0; c < n; ++c)
          if (nw[c] >= keep_min && nw[c] > 0.0 && mx > 0.0) {
            idx.push_back(c);
            if (equilibrate) scale[(size_t)w * nmax + c] = 1.0 / nw[c];
          }
        // largest norm first; ties keep their column order
        std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return nw[x] > nw[y]; });
        n2[w] = (int)idx.size();
        if (n2[w] < 1) { bad[w] = 1; continue; }
        if (n2[w] > in[w].m) { bad[w] = 2; continue; }
        std::copy(idx.begin(), idx.end(), perm.begin() + (size_t)w * nmax);
      } catch (const std::bad_alloc &) {
        bad[w] = 3;
      }
    }
  };
  const int nth = W >= 256 ? (int)std::min(16u, std::max(1u, std::thread::hardware_concurrency())) : 1;
  if (nth == 1) {
    select(0, W);
  } else {
    std::vector<std::thread> th;
    const int per = cdiv(W, nth);
    for (int w0 = 0; w0 < W; w0 += per) th.emplace_back(select, w0, std::min(W, w0 + per));
    for (auto &t : th) t.join();
  }
  for (int w = 0; w < W; ++w) {
    MFS_REQUIRE(bad[w] != 1, "graded pseudoinverse: matrix is zero");
    MFS_REQUIRE(bad[w] != 2, "graded pseudoinverse: more independent columns than rows");
    if (bad[w] == 3) MFS_THROW(MFS_ENOMEM, "graded pseudoinverse: out of host memory ordering the columns");
  }
  g.perm.alloc(perm.size() * sizeof(int));
  HIP_CHECK(hipMemcpyAsync(g.perm.p, perm.data(), perm.size() * sizeof(int), hipMemcpyHostToDevice, s));
  g.colscale.release();
  if (equilibrate) {
    g.colscale.alloc(scale.size() * sizeof(double));
    HIP_CHECK(hipMemcpyAsync(g.colscale.p, scale.data(), scale.size() * sizeof(double), hipMemcpyHostToDevice, s));
    HIP_CHECK(hipStreamSynchronize(s));   // `scale` goes out of scope
  }
  const double *cscl = equilibrate ? g.colscale.as<double>() : nullptr;
  const int n2max = *std::max_element(n2.begin(), n2.end());
  int nwhole = n2max;   // columns of the widest whole matrix
  for (int w = 0; halves && w < W; w += 2) nwhole = std::max(nwhole, n2[w] + n2[w + 1]);
  // 2. QR without pivoting of the selected, ordered columns
  g.h_qc.resize(W);
  g.small.alloc((size_t)4 * W * sizeof(int));
  int *flags = g.small.as<int>();
  // one allocation per kind for the whole batch (a matrix's pieces at 256-byte
  // aligned offsets): thousands of matrices cost no allocation each
  std::vector<size_t> oa(W), of(W);
  // panel width of the blocked QR of the ordered columns, measured for this
  // size class (qr_tuned_nb)
  // Cholesky panels where the columns are expected to be independent
  const bool chol = equilibrate && chol_panels();
  g.qr_nb = qr_tuned_nb(in, s, chol);
  const int nbq = g.qr_nb;
  {
    size_t ta = 0, tf = 0;
    for (int w = 0; w < W; ++w) {
      const int ldq = in[w].lda, n = n2[w], npan = cdiv(n, nbq);
      oa[w] = ta;
      ta += arena_bytes((size_t)ldq * n);
      of[w] = tf;
      tf += arena_bytes((size_t)n + (size_t)npan * nbq * nbq + (size_t)ldq * n);
    }
    g.qc_a.alloc(ta);
    g.qc_fac.alloc(tf);
  }
  for (int w = 0; w < W; ++w) {
    const int m = in[w].m, ldq = in[w].lda, n = n2[w];
    const int npan = cdiv(n, nbq);
    MatDesc d{};
    double2 *p = arena_at(g.qc_fac, of[w]);
    d.a = arena_at(g.qc_a, oa[w]); d.m = m; d.n = n; d.lda = ldq;
    d.tau = p; p += n;
    d.T = p; p += (size_t)npan * nbq * nbq;
    d.u = p;
    d.rank = flags + W + w;       // shared with the Jacobi descriptor (kept rank)
    g.h_qc[w] = d;
  }
  upload_descs(g.d_qc, g.h_qc, s);
  hipLaunchKernelGGL(gather_kernel, dim3(n2max, W), dim3(256), 0, s, g.d_in.as<MatDesc>(), g.d_qc.as<MatDesc>(),
                     g.perm.as<int>(), nmax, cscl, nullptr);
  HIP_CHECK(hipGetLastError());
  EvPair qre(s);
  g.redone = 0;
  if (chol) {
    DevBuf bad((size_t)cdiv(W, 4) * sizeof(double2));
    launch_zero(bad.as<double2>(), cdiv(W, 4), s);
    qr_factor(g.d_qc.as<MatDesc>(), g.h_qc, s, nbq, bad.as<int>());
    std::vector<int> hb(W);
    HIP_CHECK(hipMemcpyAsync(hb.data(), bad.p, W * sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    // the matrices with nearly dependent columns again by column steps (each
    // on its own verdict, whatever the other waves' are)
    std::vector<MatDesc> redo;
    for (int w = 0; w < W; ++w)
      if (hb[w]) redo.push_back(g.h_qc[w]);
    g.redone = (int)redo.size();
    if (!redo.empty()) {
      hipLaunchKernelGGL(gather_kernel, dim3(n2max, W), dim3(256), 0, s, g.d_in.as<MatDesc>(), g.d_qc.as<MatDesc>(),
                         g.perm.as<int>(), nmax, cscl, bad.as<int>());
      DevBuf dr;
      upload_descs(dr, redo, s);
      qr_factor(dr.as<MatDesc>(), redo, s, nbq);
      HIP_CHECK(hipStreamSynchronize(s));
    }
  } else {
    qr_factor(g.d_qc.as<MatDesc>(), g.h_qc, s, nbq);
  }
  qre.stop(s);
  if (g.ev_qr_done) HIP_CHECK(hipEventRecord(g.ev_qr_done, s));
  g.qr_flops = 0.0;
  for (int w = 0; w < W; ++w) {
    const double m = in[w].m, n = n2[w];
    g.qr_flops += 8.0 * m * n * n - 8.0 * n * n * n / 3.0;
  }
  EvPair poste(s);
  struct Finish {   // the QR and post-QR times, however graded_pinv returns
    GradedPinv &g; EvPair &a, &b; hipStream_t s;
    ~Finish() {
      b.stop(s);
      if (hipStreamSynchronize(s) == hipSuccess) { g.qr_ms = a.ms(); g.post_ms = b.ms(); }
    }
  } fin{g, qre, poste, s};
  // the triangle that the row selection and the LQ read: R from the
  // column-pivoted QR R_1 P_2 = Q_2 R (its rows carry the grading, which the
  // right factor from L^{-1} rests on)
  {
    std::vector<int> ident((size_t)W * nmax);
    for (int w = 0; w < W; ++w)
      for (int i = 0; i < nmax; ++i) ident[(size_t)w * nmax + i] = i;
    g.piv.alloc(ident.size() * sizeof(int));
    HIP_CHECK(hipMemcpyAsync(g.piv.p, ident.data(), ident.size() * sizeof(int), hipMemcpyHostToDevice, s));
    HIP_CHECK(hipStreamSynchronize(s));
  }
  if (equilibrate && direct_pinv(g, n2, nmax, rel_cutoff, cscl, in, s, keep_reflectors, halves)) return;
  {
    g.h_rq.resize(W);
    {
      size_t ta = 0, tf = 0;
      for (int w = 0; w < W; ++w) {
        const int n = n2[w], ldr = round_up(n, 16), npan = cdiv(n, kQRNB);
        oa[w] = ta;
        ta += arena_bytes((size_t)ldr * n);
        of[w] = tf;
        tf += arena_bytes((size_t)n + (size_t)npan * kQRNB * kQRNB);
      }
      g.rq_a.alloc(ta);
      g.rq_fac.alloc(tf);
    }
    for (int w = 0; w < W; ++w) {
      const int n = n2[w], ldr = round_up(n, 16);
      MatDesc d{};
      double2 *p = arena_at(g.rq_fac, of[w]);
      d.a = arena_at(g.rq_a, oa[w]); d.m = n; d.n = n; d.lda = ldr;
      d.tau = p; p += n;
      d.T = p;
      d.rank = flags + W + w;
      g.h_rq[w] = d;
    }
    upload_descs(g.d_rq, g.h_rq, s);
    hipLaunchKernelGGL(copy_r_kernel, dim3(1024, W), dim3(256), 0, s, g.d_qc.as<MatDesc>(), g.d_rq.as<MatDesc>());
    HIP_CHECK(hipGetLastError());
    // From 256 columns on, and in large batches, the pivots of each 32-column
    // block are chosen on a Gaussian sketch (qrcp_sketch.hip): A is read once per
    // block, not per column (the large periodizer's 8 triangles of 10805 columns:
    // 7.3 -> 3.0 s per incidence; the 256-obstacle batch's triangles: truncation
    // 10.3 -> 8.8 s).  Below, they are the columns of largest remaining norm: a
    // sketch gains nothing there (33 triangles of 200 columns 9.9 ms a pass from
    // the geometry with either, of 250 13.6 and 13.9), and its pivots are not the
    // norms'; the fields' errors against 64 bits are the same on average over 14
    // bodies of 129 to 242 columns, but 8.9e-15 sketched and 6.9e-15 not for the
    // k = 10 body, 1.5e-14 and 0.96e-14 for 13 of 220 columns.  Triangles that
    // fit a workgroup's registers take one launch with a workgroup a matrix
    // (qrcp_one_kernel: a penetrable body's 17 of 120 columns 3.7 ms a pass, 4.3
    // sketched), the others two launches a column over the whole chip.
    // MFS_QRCP=sketched, unblocked (two launches a column) or blocked (panels of
    // 32, updates deferred, norms downdated, qrcp.hip) decides.
    const char *qe = std::getenv("MFS_QRCP");
    const bool big = n2max >= 256 || (size_t)W * n2max * n2max >= ((size_t)1 << 24);
    const std::string form = qe ? std::string(qe) : (big ? "sketched" : n2max <= QN ? "one" : "unblocked");
    DevBuf qn;   // column norms, where the form reads them
    if (form != "sketched" && !(form == "one" && n2max <= QN)) {
      qn.alloc((size_t)W * nmax * sizeof(double));
      hipLaunchKernelGGL(colnorm_kernel, dim3(cdiv(n2max, 4), W), dim3(256), 0, s, g.d_rq.as<MatDesc>(),
                         qn.as<double>(), nmax);
    }
    if (form == "one" && n2max <= QN) {
      if (n2max <= 64)
        hipLaunchKernelGGL((qrcp_one_kernel<1, 4>), dim3(W), dim3(64 * QW), 0, s, g.d_rq.as<MatDesc>(),
                           g.piv.as<int>(), nmax);
      else
        hipLaunchKernelGGL((qrcp_one_kernel<2, 8>), dim3(W), dim3(64 * QW), 0, s, g.d_rq.as<MatDesc>(),
                           g.piv.as<int>(), nmax);
    } else if (form == "sketched") {
      qrcp_sketched(g.d_rq.as<MatDesc>(), g.h_rq, g.piv.as<int>(), nmax, s);
    } else if (form != "blocked") {
      for (int k = 0; k < n2max; ++k) {
        hipLaunchKernelGGL(qrcp_pivot_kernel, dim3(W), dim3(PK), 0, s, g.d_rq.as<MatDesc>(), k, qn.as<double>(),
                           g.piv.as<int>(), nmax);
        if (k + 1 < n2max)
          hipLaunchKernelGGL(qrcp_update_kernel, dim3(cdiv(n2max - k - 1, 4), W), dim3(256), 0, s,
                             g.d_rq.as<MatDesc>(), k, qn.as<double>(), nmax);
      }
    } else {
      qrcp_blocked(g.d_rq.as<MatDesc>(), g.h_rq, qn.as<double>(), g.piv.as<int>(), nmax, s);
    }
    HIP_CHECK(hipGetLastError());
    // T of 32-column panels: read where U is formed with panels that narrow
    // only (qr_form_u regroups wider matrices into 64 columns)
    if (n2max <= kQRNB)
      hipLaunchKernelGGL(build_t_kernel, dim3(W, cdiv(n2max, kQRNB)), dim3(256), 0, s, g.d_rq.as<MatDesc>());
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(s));   // qn is released here
  }
  const MatDesc *tri = g.d_rq.as<MatDesc>();
  // rows of the triangle to keep
  DevBuf rn((size_t)W * n2max * sizeof(double));
  hipLaunchKernelGGL(rownorm_kernel, dim3(cdiv(n2max, 256), W), dim3(256), 0, s, tri, rn.as<double>(), n2max);
  HIP_CHECK(hipGetLastError());
  std::vector<double> hr((size_t)W * n2max);
  HIP_CHECK(hipMemcpyAsync(hr.data(), rn.p, hr.size() * sizeof(double), hipMemcpyDeviceToHost, s));
  HIP_CHECK(hipStreamSynchronize(s));
  for (int w = 0; w < W; ++w) {
    const double thr = 1e-15 * g.maxcol[w];
    double suf = 0.0;
    int r = n2[w];
    for (int i = n2[w] - 1; i >= 0; --i) {
      suf += hr[(size_t)w * n2max + i];
      if (std::sqrt(suf) > thr) { r = i + 1; break; }
      r = i;
    }
    rr[w] = std::max(r, 1);
  }
  // complete orthogonal decomposition: keep the rows of the pivoted triangle
  // until the trailing block's Frobenius norm is at most rel_cutoff times the
  // largest singular value (the rank-revealing counterpart of the SVD cut)
  const bool cod = use_cod(equilibrate, nwhole);
  g.cod = cod;
  if (cod) {
    std::vector<double> s1 = tri_sigma1(tri, n2, n2max, s);
    for (int w = 0; halves && w < W; w += 2) s1[w] = s1[w + 1] = std::max(s1[w], s1[w + 1]);
    for (int w = 0; w < W; ++w) {
      const double thr = rel_cutoff * s1[w];
      double suf = 0.0;
      int r = rr[w];
      for (int i = rr[w] - 1; i >= 0; --i) {
        suf += hr[(size_t)w * n2max + i];
        if (std::sqrt(suf) > thr) { r = i + 1; break; }
        r = i;
      }
      rr[w] = std::max(r, 1);
    }
  }
  g.rows = rr;
  g.cols = n2;
  // 3. QR of R_top^H (n2 x r)  and  4. Jacobi on L = (R factor)^H
  g.h_lq.resize(W);
  {
    size_t ta = 0, tf = 0;
    for (int w = 0; w < W; ++w) {
      const int m = n2[w], n = rr[w];
      const int ld2 = round_up(m, 16), ldg = round_up(n, 16), npan = cdiv(n, kQRNB);
      oa[w] = ta;
      ta += arena_bytes((size_t)ld2 * n);
      of[w] = tf;
      // tau, T, g, u, then sv and perm (2 n doubles' worth)
      tf += arena_bytes((size_t)n + (size_t)npan * kQRNB * kQRNB + (size_t)n * ldg + (size_t)ld2 * n + n);
    }
    g.lq_a.alloc(ta);
    g.lq_fac.alloc(tf);
  }
  for (int w = 0; w < W; ++w) {
    const int m = n2[w], n = rr[w];
    const int ld2 = round_up(m, 16), ldg = round_up(n, 16);
    const int npan = cdiv(n, kQRNB);
    double2 *p = arena_at(g.lq_fac, of[w]);
    MatDesc d{};
    d.a = arena_at(g.lq_a, oa[w]); d.m = m; d.n = n; d.lda = ld2;
    d.tau = p; p += n;
    d.T = p; p += (size_t)npan * kQRNB * kQRNB;
    d.g = p; p += (size_t)n * ldg;
    d.u = p; p += (size_t)ld2 * n;
    d.ldg = ldg;
    double *rp = reinterpret_cast<double *>(p);
    d.sv = rp;
    d.perm = reinterpret_cast<int *>(rp + n);
    d.rank = flags + W + w;
    g.h_lq[w] = d;
  }
  upload_descs(g.d_lq, g.h_lq, s);
  hipLaunchKernelGGL(transpose_top_kernel, dim3(1024, W), dim3(256), 0, s, tri, g.d_lq.as<MatDesc>());
  HIP_CHECK(hipGetLastError());
  qr_factor(g.d_lq.as<MatDesc>(), g.h_lq, s);
  const int rmax = *std::max_element(rr.begin(), rr.end());
  if (cod) {
    // every kept row stays: L^{-1} = (R_L^{-1})^H in place of V_L S^+, U_L = I
    g.kept = rr;
    g.jacobi_ms = g.jacobi_bytes = g.jacobi_flops = 0.0;
    g.jacobi_launches = 0;
    g.jacobi_unconverged = 0;
    HIP_CHECK(hipMemcpyAsync(flags + W, rr.data(), W * sizeof(int), hipMemcpyHostToDevice, s));
  } else {
    const JacStats js = jac_run(g.d_lq.as<MatDesc>(), g.h_lq, 1, rel_cutoff, s);
    g.jacobi_ms = js.ms;
    g.jacobi_launches = js.launches;
    g.jacobi_bytes = js.bytes;
    g.jacobi_flops = js.flops;
    g.jacobi_unconverged = js.unconverged;
    jac_sort(g.d_lq.as<MatDesc>(), g.h_lq, rel_cutoff, s, g.kept, halves);
  }
  // X = R_L^{-1}, for L^{-1} (decomposition) or V_L S^+ = L^{-1} U_L
  DevBuf xa, dx;
  {
    std::vector<size_t> ox(W);
    size_t tx = 0;
    for (int w = 0; w < W; ++w) {
      ox[w] = tx;
      tx += arena_bytes((size_t)round_up(rr[w], 16) * rr[w]);
    }
    xa.alloc(tx);
    std::vector<MatDesc> hx(W);
    for (int w = 0; w < W; ++w) {
      MatDesc d{};
      d.a = arena_at(xa, ox[w]);
      d.m = rr[w]; d.n = rr[w]; d.lda = round_up(rr[w], 16);
      d.rank = flags + W + w;
      hx[w] = d;
    }
    upload_descs(dx, hx, s);
    launch_zero(xa.as<double2>(), (long)(tx / sizeof(double2)), s);
    const int nblk = cdiv(rmax, TI);
    hipLaunchKernelGGL(trinv_diag_kernel, dim3(nblk, W), dim3(256), 0, s, g.d_lq.as<MatDesc>(), dx.as<MatDesc>());
    trinv_offdiag(g.d_lq.as<MatDesc>(), dx.as<MatDesc>(), W, nblk, s);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(s));   // hx goes out of scope
  }
  // 5. explicit factors
  int kmax = 0;
  for (int k : g.kept) kmax = std::max(kmax, k);
  if (cod)
    hipLaunchKernelGGL(cod_prep_kernel, dim3(rmax, W), dim3(256), 0, s, g.d_qc.as<MatDesc>(),
                       g.d_lq.as<MatDesc>(), dx.as<MatDesc>());
  else {
    hipLaunchKernelGGL(prep_u_kernel, dim3(rmax, W), dim3(256), 0, s, g.d_qc.as<MatDesc>(), g.d_lq.as<MatDesc>());
    if (kmax > 0)
      hipLaunchKernelGGL(right_factor_kernel, dim3(cdiv(kmax, 64), cdiv(rmax, 64), W), dim3(256), 0, s,
                         g.d_lq.as<MatDesc>(), dx.as<MatDesc>());
  }
  HIP_CHECK(hipGetLastError());
  // U = Q_1 [Q_2 [U_L; 0]; 0] (the reflectors of the pivoted triangle act on
  // the first n2 rows first); V = Z V_L, before the column orders are undone in W
  {
    g.h_rqu = g.h_rq;
    for (int w = 0; w < W; ++w) {
      g.h_rqu[w].u = g.h_qc[w].u;
      g.h_rqu[w].ldu = g.h_qc[w].lda;
    }
    upload_descs(g.d_rqu, g.h_rqu, s);
    qr_form_u(g.d_rqu.as<MatDesc>(), g.h_rqu, kmax, s);
  }
  qr_form_u(g.d_qc.as<MatDesc>(), g.h_qc, kmax, s, false, nbq);
  qr_form_u(g.d_lq.as<MatDesc>(), g.h_lq, kmax, s);
  g.h_fin.resize(W);
  {
    size_t tf = 0;
    for (int w = 0; w < W; ++w) {
      of[w] = tf;
      tf += arena_bytes((size_t)round_up(in[w].n, 16) * std::max(1, g.kept[w]));
    }
    g.fin_w.alloc(tf);
  }
  for (int w = 0; w < W; ++w) {
    const int n = in[w].n, ldw = round_up(n, 16);
    MatDesc d{};
    d.m = in[w].m; d.n = n; d.lda = g.h_qc[w].lda;
    d.u = g.h_qc[w].u;
    d.w = arena_at(g.fin_w, of[w]);
    d.ldg = ldw;
    d.rank = flags + W + w;
    g.h_fin[w] = d;
  }
  upload_descs(g.d_fin, g.h_fin, s);
  if (kmax > 0) {
    hipLaunchKernelGGL(scatter_w_kernel, dim3(kmax, W), dim3(256), 0, s, g.d_lq.as<MatDesc>(), g.d_fin.as<MatDesc>(),
                       g.perm.as<int>(), g.piv.as<int>(), nmax, cscl);
    HIP_CHECK(hipGetLastError());
  }
  HIP_CHECK(hipStreamSynchronize(s));
}

void GradedPinv::singular_values(int ldo, std::vector<double> &out, hipStream_t s) const {
  const int W = (int)h_lq.size();
  out.assign((size_t)W * ldo, 0.0);
  if (W == 0 || ldo <= 0 || cod) return;   // the decomposition forms no singular values
  DevBuf buf(out.size() * sizeof(double));
  hipLaunchKernelGGL(sv_gather_kernel, dim3(W), dim3(256), 0, s, d_lq.as<MatDesc>(), ldo, buf.as<double>());
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipMemcpyAsync(out.data(), buf.p, out.size() * sizeof(double), hipMemcpyDeviceToHost, s));
  HIP_CHECK(hipStreamSynchronize(s));
}

}  // namespace mfs
