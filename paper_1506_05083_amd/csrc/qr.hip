// Batched blocked Householder QR of tall complex matrices (the dense
// least-squares factorisations of Sec. 3, eq. (linsys), and of the
// periodizing matrix Q of Sec. 4.2), LAPACK's zlarfg convention:
// H = I - tau v v^H, v(1) = 1, H^H x = beta e_1 with beta real.
//
// Panels of 16 columns, in one launch while a panel's rows fit a workgroup
// (bqr_panel_kernel), by Cholesky QR where the caller's columns are independent
// (cq_* kernels), else column by column with one launch per column that spans all
// rows of all matrices (CH-row chunks, one row per thread, the row's panel entries
// in registers):
//   * launch s finishes reflector s from the chunk partial sums written by
//     launch s-1: |x(2:)|^2 and x^H a_c for the panel columns c > s (so the
//     reflector and every w_c = v^H a_c follow from one pass over the rows),
//     with row j of the panel read from a side buffer that no workgroup of
//     launch s writes;
//   * it then applies H_s^H to its rows of the columns c > s and writes the
//     partial sums of step s + 1.
// The trailing matrix is updated with the compact-WY form
// C <- (I - V T V^H)^H C = C - V T^H (V^H C):
//   bqr_vhy_kernel   P = V^H [V | C], split over row slices (partials);
//   bqr_t_kernel     T from the V^H V part (forward, columnwise);
//   bqr_w2_kernel    W2 = op(T) (V^H C), the slices summed;
//   bqr_update       C -= V W2 on the matrix cores.
// The same three apply kernels with T in place of T^H, run over the panels
// in reverse, form U = Q [U_R; 0] for the explicit left singular vectors.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>

#include "internal.hpp"

namespace mfs {
namespace {

constexpr int CH = 256;     // rows per workgroup in the panel column step
constexpr int KRMIN = 64;   // fewest rows of a V^H Y split-K slice
constexpr int KS = 16;      // rows per LDS stage in V^H Y
// V^H Y tiles: YT columns of Y a workgroup, a wave IB x CB blocks of 16 x 16
// of the NB x YT tile, OCC waves a SIMD, DB: LDS stages double-buffered (one
// barrier a stage), KR rows a workgroup (one split-K slice: each slice writes
// an NB-row partial of P that W2 and T read back).  Measured on 8 matrices
// 4608 x 1275 with 256-row slices: 64-column panels 54 TFLOP/s (43 with one
// 16-row block of V^H and four column blocks a wave and the fragments loaded
// per product), 32: 43 (33), 16: 3.8 TB/s of Y.  The 64-wide panels take
// 512-row slices: on that shape V^H Y is 8% slower and W2 as much faster, on
// the 25088-row Q of the large cup the QR and U formation gain 2%.
template <int NB> struct VhyShape;
template <> struct VhyShape<64> { static constexpr int YT = 64, IB = 2, CB = 2, OCC = 2, DB = 0, KR = 512; };
template <> struct VhyShape<32> { static constexpr int YT = 64, IB = 1, CB = 2, OCC = 3, DB = 1, KR = 256; };
template <> struct VhyShape<16> { static constexpr int YT = 64, IB = 1, CB = 1, OCC = 4, DB = 1, KR = 256; };
constexpr int W2T = 16;     // columns per W2 tile (the slices' sum spread over more workgroups)
constexpr int W2WG = 8192;  // workgroups a W2 launch aims at; beyond it a workgroup takes several tiles

// element r of Householder vector i of the panel starting at column k0
__device__ inline double2 vel(const MatDesc &d, int k0, int i, int r) {
  const int c = k0 + i;
  const double2 x = ld_or0(d.a, (size_t)c * d.lda + r, c < d.n && r > c && r < d.m);
  return csel(c < d.n && r == c, cz(1.0, 0.0), x);
}

__device__ inline int ldu_of(const MatDesc &d) { return d.ldu ? d.ldu : d.lda; }

// Panel column step s (s = -1: partial sums of step 0 only).
// part: [mat][2][nchmax][NPART] (slot [0].x: |x(2:)|^2, slot 1 + c: x^H a_c)
// side: [mat][2][NB] row j of the panel columns
template <int NB>
__global__ __launch_bounds__(CH) void bqr_col_kernel(const MatDesc *__restrict__ descs, int k0, int s,
                                                     double2 *__restrict__ part, double2 *__restrict__ side,
                                                     int nchmax) {
  constexpr int NPART = NB + 1;
  constexpr int SUB = CH / NPART;   // threads per slot summing the chunk partials
  static_assert(SUB >= 1, "a column-step workgroup sums every partial slot");
  const MatDesc d = descs[blockIdx.y];
  if (k0 >= d.n) return;
  const int nbp = min(NB, d.n - k0);
  if (s >= nbp) return;
  const int mrows = d.m - k0;
  if ((int)blockIdx.x * CH >= mrows) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int r = k0 + blockIdx.x * CH + tid;
  const bool live = r < d.m;
  double2 *pb = part + (size_t)blockIdx.y * 2 * nchmax * NPART;
  double2 *sb = side + (size_t)blockIdx.y * 2 * NB;
  __shared__ double2 fin[NPART];
  __shared__ double2 fsum[NPART][SUB];
  __shared__ double2 sf[NB];
  __shared__ double2 red[CH / 64][NPART];
  __shared__ double2 s_scale, s_tau, s_alpha;
  __shared__ double s_beta;
  __shared__ int s_refl;

  double2 vals[NB];
  const int cfirst = s < 0 ? 0 : s;
#pragma unroll
  for (int c = 0; c < NB; ++c)
    vals[c] = ld_or0(d.a, (size_t)(k0 + c) * d.lda + r, live && c >= cfirst && c < nbp);

  if (s >= 0) {
    const int j = k0 + s;
    const double2 *pin = pb + (size_t)(s & 1) * nchmax * NPART;
    const double2 *srow = sb + (s & 1) * NB;
    const int nch = (mrows + CH - 1) / CH;
    // chunk partials summed by SUB threads per slot, then across them
    if (tid < NPART * SUB) {
      const int slot = tid / SUB, sub = tid % SUB;
      double2 t = cz(0.0, 0.0);
      for (int ch = sub; ch < nch; ch += SUB) t = cadd(t, pin[(size_t)ch * NPART + slot]);
      fsum[slot][sub] = t;
    }
    __syncthreads();
    if (tid < NPART) {
      double2 t = fsum[tid][0];
#pragma unroll
      for (int u = 1; u < SUB; ++u) t = cadd(t, fsum[tid][u]);
      fin[tid] = t;
    }
    __syncthreads();
    if (tid == 0) {
      const double ssum = fin[0].x;
      const double2 alpha = srow[s];
      s_alpha = alpha;
      if (ssum == 0.0 && alpha.y == 0.0) {
        s_refl = 0;
        s_tau = cz(0.0, 0.0);
        s_beta = alpha.x;
        s_scale = cz(0.0, 0.0);
      } else {
        const double beta = -copysign(sqrt(alpha.x * alpha.x + alpha.y * alpha.y + ssum), alpha.x);
        const double2 den = cz(alpha.x - beta, alpha.y);
        const double dd = cabs2(den);
        s_refl = 1;
        s_tau = cz((beta - alpha.x) / beta, -alpha.y / beta);
        s_beta = beta;
        s_scale = cz(den.x / dd, -den.y / dd);
      }
      if (blockIdx.x == 0) d.tau[j] = s_tau;
    }
    __syncthreads();
    const double2 scale = s_scale, tau = s_tau, alpha = s_alpha;
    const int refl = s_refl;
    if (tid > s && tid < nbp) {
      // w_c = v^H a_c = a_c(j) + conj(scale) (x^H a_c - conj(alpha) a_c(j))
      const double2 acj = srow[tid];
      double2 w = fin[1 + tid];
      w = csub(w, cmul(cconj(alpha), acj));
      w = cadd(acj, cmul(cconj(scale), w));
      sf[tid] = refl ? cmul(cconj(tau), w) : cz(0.0, 0.0);
    }
    __syncthreads();
    double2 xs = cz(0.0, 0.0);   // vals[s] without a run-time index into the array
#pragma unroll
    for (int c = 0; c < NB; ++c)
      if (c == s) xs = vals[c];
    if (live && r >= j) {
      double2 v;
      if (r == j) {
        v = cz(1.0, 0.0);
        d.a[(size_t)j * d.lda + j] = refl ? cz(s_beta, 0.0) : alpha;
      } else {
        v = refl ? cmul(xs, scale) : xs;
        d.a[(size_t)j * d.lda + r] = v;
      }
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        if (c > s && c < nbp) {
          vals[c] = csub(vals[c], cmul(v, sf[c]));
          d.a[(size_t)(k0 + c) * d.lda + r] = vals[c];
        }
      }
    }
  }

  // partial sums of step s + 1
  const int s1 = s + 1;
  if (s1 >= nbp) return;
  const int j1 = k0 + s1;
  double2 x = cz(0.0, 0.0);
#pragma unroll
  for (int c = 0; c < NB; ++c)
    if (c == s1) x = vals[c];
  if (!(live && r >= j1)) x = cz(0.0, 0.0);
  if (live && r == j1) {
#pragma unroll
    for (int c = 0; c < NB; ++c)
      if (c >= s1 && c < nbp) sb[(s1 & 1) * NB + c] = vals[c];
  }
  double2 *pout = pb + (size_t)(s1 & 1) * nchmax * NPART + (size_t)blockIdx.x * NPART;
  {
    double q = (live && r > j1) ? cabs2(x) : 0.0;
    q = wave_sum(q);
    if (lane == 0) red[wv][0] = cz(q, 0.0);
  }
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    if (c > s1 && c < nbp) {
      double2 p = cz(0.0, 0.0);
      cfmac(p, x, vals[c]);
      p = wave_sum(p);
      if (lane == 0) red[wv][1 + c] = p;
    }
  }
  __syncthreads();
  if (tid < NPART && (tid == 0 || (tid - 1 > s1 && tid - 1 < nbp))) {
    double2 t = red[0][tid];
#pragma unroll
    for (int w = 1; w < CH / 64; ++w) t = cadd(t, red[w][tid]);
    pout[tid] = t;
  }
}

// The whole panel at k0 of a matrix whose rows from k0 on fit one workgroup
// (m - k0 <= PTMAX) in one launch, with the panel's T.  A thread holds one
// column c = lane % 16 of the rows 4 u + lane / 16 (u < RPT) of its wave's
// 4 RPT rows, wave 0 the first.  Step S:
//   * column S goes from lane S to its row of 16 lanes by DPP, and every thread
//     adds up t_c = sum conj(x_r) a_c(r) over its rows r below j = k0 + S;
//     the four threads of a column in a wave are added by lane swaps, the
//     waves through LDS (one barrier a step, two buffers);
//   * t_S = |x(2:)|^2 gives LAPACK's zlarfg reflector v = scale x (1 on row j),
//     w_c = v^H a_c = a_c(j) + conj(scale) t_c, and the columns c > S are
//     updated: a_c(r) -= x_r (scale tau^* w_c), row j by tau^* w_c;
//   * the finished columns c < S hold x unscaled, so their t_c is what
//     v_c^H v_S of T needs.
// The columns are scaled to v at the end, and wave 0 runs T's recurrence.
// A step is a serial chain (sums, square root, division, update).  With a row a
// thread, every column's sum a DPP scan of its own and five barriers, a step
// took 4 us whatever the rows: 17 panels of 60 rows 50 -> 19 us, 65 of 250 rows
// 67 -> 31, and 65 of 700 rows, a launch a column, 144 -> 55.  Past PTMAX rows the
// entries no longer fit a workgroup's registers.
constexpr int PTMAX = 1024;   // rows of the one-launch panel
constexpr int PNB = 16;       // its columns

// sum over the wave's four rows of 16 lanes, the same bits in all of them
__device__ inline double sum_rows16(double v) {
  v = swap16_add(v, v);
  return swap32_add(v, v);
}

struct PanelShared {
  double2 red[2][PTMAX / 64][PNB], row[2][PNB];
  double2 g[PNB][PNB + 1], tau[PNB];
};

template <int S, int RPT, int NWMAX>
__device__ inline void panel_steps(double2 (&a)[RPT], double2 &myscale, PanelShared &sh, int nbp,
                                   int wv, int c, int k) {
  if constexpr (S < PNB) {
    if (S < nbp) {   // uniform
      constexpr int B = S & 1, U = S / 4;
      const bool top = wv == 0;
      double2 t = cz(0.0, 0.0), t1 = t;
#pragma unroll
      for (int u = 0; u < RPT; ++u) {
        // the rows in order: fetched ahead, x takes 4 RPT registers
        if (u >= 2) asm volatile("" : "+v"(a[u].x), "+v"(a[u].y) : "v"(t.x), "v"(t1.x));
        double2 x = row_lane<S>(a[u]);
        if (u <= U) x = csel(top && 4 * u + k <= S, cz(0.0, 0.0), x);
        cfmac((u & 1) ? t1 : t, x, a[u]);
      }
      t = cadd(t, t1);
      t = cz(sum_rows16(t.x), sum_rows16(t.y));
      if (k == 0) sh.red[B][wv][c] = t;
      if (top && k == (S & 3)) sh.row[B][c] = a[U];
      __syncthreads();
      t = cz(0.0, 0.0);
#pragma unroll
      for (int w = 0; w < NWMAX; w += 4) t = cadd(t, sh.red[B][w + k][c]);   // 0 past the last wave
      t = cz(sum_rows16(t.x), sum_rows16(t.y));
      const double2 acj = sh.row[B][c], alpha = sh.row[B][S];
      const double ssum = row_lane<S>(t.x);
      double2 tau = cz(0.0, 0.0), scale = cz(0.0, 0.0), diag = alpha;
      if (!(ssum == 0.0 && alpha.y == 0.0)) {
        const double beta = -copysign(sqrt(alpha.x * alpha.x + alpha.y * alpha.y + ssum), alpha.x);
        const double2 den = cz(alpha.x - beta, alpha.y);
        const double dd = cabs2(den);
        tau = cz((beta - alpha.x) / beta, -alpha.y / beta);
        scale = cz(den.x / dd, -den.y / dd);
        diag = cz(beta, 0.0);
      }
      // tau^* (a_c(j) + conj(scale) t_c) of the columns still to come
      double2 f = acj;
      cfma(f, cconj(scale), t);
      f = csel(c > S, cmul(cconj(tau), f), cz(0.0, 0.0));
      const double2 g = cmul(scale, f), mg = cz(-g.x, -g.y);
      if (top && k == 0 && c < S)   // v_c^H v_S
        sh.g[c][S] = cmul(cconj(myscale), cadd(cconj(acj), cmul(scale, cconj(t))));
#pragma unroll
      for (int u = 0; u < RPT; ++u) {
        // likewise, and column S fetched again rather than kept from above
        if (u >= 2)
          asm volatile("" : "+v"(a[u].x), "+v"(a[u].y) : "v"(a[u - 2].x), "v"(a[u - 2].y));
        else
          asm volatile("" : "+v"(a[u].x), "+v"(a[u].y) : "v"(mg.x));
        double2 x = row_lane<S>(a[u]);
        if (u <= U) x = csel(top && 4 * u + k <= S, cz(0.0, 0.0), x);
        cfma(a[u], x, mg);
      }
      if (top && k == (S & 3)) a[U] = c == S ? diag : csub(a[U], f);
      myscale = csel(c == S, scale, myscale);
      if (top && c == 0 && k == 0) sh.tau[S] = tau;
      panel_steps<S + 1, RPT, NWMAX>(a, myscale, sh, nbp, wv, c, k);
    }
  }
}

// row c of T = -T V^H V tau, upper triangular, a column at a time
template <int S>
__device__ inline void panel_t(double2 (&t)[PNB], double2 mytau, const PanelShared &sh, int nbp, int c) {
  if constexpr (S < PNB) {
    const double2 tau = row_lane<S>(mytau);
    double2 acc = cz(0.0, 0.0);
    if (S < nbp) {
#pragma unroll
      for (int i = 0; i < S; ++i) cfma(acc, t[i], sh.g[i][S]);
    }
    acc = cmul(cz(-tau.x, -tau.y), acc);
    t[S] = S >= nbp || c > S ? cz(0.0, 0.0) : csel(c == S, tau, acc);
    panel_t<S + 1>(t, mytau, sh, nbp, c);
  }
}

template <int RPT, int NWMAX>
__global__ __launch_bounds__(64 * NWMAX) void bqr_panel_kernel(const MatDesc *__restrict__ descs, int k0, int nbo,
                                                               double2 *__restrict__ tx) {
  const MatDesc d = descs[blockIdx.x];
  if (k0 >= d.n) return;
  const int nbp = min(PNB, d.n - k0);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int c = lane & 15, k = lane >> 4;
  __shared__ PanelShared sh;
  for (int i = tid; i < 2 * (PTMAX / 64) * PNB; i += blockDim.x) (&sh.red[0][0][0])[i] = cz(0.0, 0.0);
  const int r0 = k0 + 4 * RPT * wv + k;
  double2 *col = d.a + (size_t)(k0 + min(c, nbp - 1)) * d.lda;
  double2 a[RPT];
#pragma unroll
  for (int u = 0; u < RPT; ++u) a[u] = ld_or0(col, r0 + 4 * u, c < nbp && r0 + 4 * u < d.m);
  double2 myscale = cz(0.0, 0.0);
  __syncthreads();
  panel_steps<0, RPT, NWMAX>(a, myscale, sh, nbp, wv, c, k);
#pragma unroll
  for (int u = 0; u < RPT; ++u) {
    const int r = r0 + 4 * u;
    if (c < nbp && r < d.m) col[r] = r > k0 + c ? cmul(a[u], myscale) : a[u];
  }
  __syncthreads();
  if (wv > 0) return;
  const double2 mytau = csel(c < nbp, sh.tau[c], cz(0.0, 0.0));
  double2 t[PNB];
  panel_t<0>(t, mytau, sh, nbp, c);
  if (k == 0) {
    if (c < nbp) d.tau[k0 + c] = mytau;
    const int o = k0 % nbo;
    double2 *T = d.T + (size_t)(k0 / nbo) * nbo * nbo + (size_t)o * nbo + o;
#pragma unroll
    for (int j = 0; j < PNB; ++j) {
      T[(size_t)j * nbo + c] = t[j];
      if (tx) tx[(size_t)blockIdx.x * PNB * PNB + j * PNB + c] = t[j];
    }
  }
}

// Panels of 16 columns by Cholesky QR with the reflectors reconstructed, for
// matrices whose columns are independent (the periodizer's equilibrated Q):
// the column steps above are a chain of 17 launches a panel, each a
// reduction over all rows (16 matrices of 2304 rows: 8.3 us a launch, most of it
// latency, 143 us a panel); this is three launches of two reductions (6, 12 and
// 16 us), and the panel's T comes with them.
//   cq_gram_kernel   G = P^H P over 256-row chunks (matrix cores);
//   cq_solve_kernel  R1 = chol(G), P <- P R1^{-1} by row-wise substitution, and
//                    the chunk sums of its Gram matrix;
//   cq_reflect_kernel R2 = chol of that (Q = P R2^{-1} is orthonormal to
//                    rounding, R = R2 R1), then LU of the top block less a
//                    unitary diagonal S, Q_top - S = L U with s_j minus the
//                    phase of the j-th pivot (Ballard, Demmel, Grigori,
//                    Jacquelin, Nguyen and Solomonik 2014), as P_top - S R2 = L W,
//                    W = U R2: V = [L; P_rest W^{-1}], tau_j = -u_jj conj(s_j),
//                    and the panel's triangle S R.  The product of the reflectors is
//                    the one whose first columns are Q S^{-1}, so T and the
//                    updates proceed as after the column steps.
// Every workgroup repeats the 16 x 16 factorisations instead of waiting for
// another launch, in a wave's registers (panel_fact; with an entry a thread, the
// step's row and column through LDS and a barrier a step the launches took 15
// and 29 us).  The substitutions are row-wise
// backward stable whatever the panel's conditioning; the orthogonality after
// the second pass needs the first Cholesky's pivots above 1e-12 of the columns'
// norms (condition below 1e6 after column scaling).  A pivot below sets the
// matrix's flag and its factors are void: the caller factors it again by
// column steps.
constexpr int CQ = 16;
constexpr double kCholPivotMin = 1e-12;

// 16 x 16 Gram matrix over the 64 rows of each wave given by ld(row of the
// wave, column), the waves' sums added through red; out[i * 16 + j]
template <class F>
__device__ inline void cq_gram(F ld, double2 (*red)[CQ * CQ], double2 *out) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c = lane & 15, k = lane >> 4;
  dx4 re = {0, 0, 0, 0}, im = re;
#pragma unroll
  for (int s0 = 0; s0 < 16; s0 += 8) {
    double2 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = ld(64 * wv + 4 * (s0 + u) + k, c);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      re = mfma_f64(x[u].x, x[u].x, re);
      re = mfma_f64(x[u].y, x[u].y, re);
      im = mfma_f64(x[u].x, x[u].y, im);
      im = mfma_f64(-x[u].y, x[u].x, im);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wv][(k + 4 * v) * CQ + c] = cz(re[v], im[v]);
  __syncthreads();
  double2 t = red[0][threadIdx.x];
#pragma unroll
  for (int w = 1; w < CH / 64; ++w) t = cadd(t, red[w][threadIdx.x]);
  out[threadIdx.x] = t;
}

__global__ __launch_bounds__(CH) void cq_gram_kernel(const MatDesc *__restrict__ descs, int k0,
                                                     double2 *__restrict__ part, int nchmax) {
  const MatDesc d = descs[blockIdx.y];
  const int r0 = k0 + blockIdx.x * CH;
  if (k0 >= d.n || r0 >= d.m) return;
  const int nbp = min(CQ, d.n - k0);
  __shared__ double2 red[CH / 64][CQ * CQ];
  cq_gram([&](int row, int c) {
    return ld_or0(d.a, (size_t)(k0 + min(c, nbp - 1)) * d.lda + min(r0 + row, d.m - 1), c < nbp && r0 + row < d.m);
  }, red, part + ((size_t)blockIdx.y * nchmax + blockIdx.x) * CQ * CQ);
}

// Sum of the chunks' Gram matrices (identity outside the nbp columns), the
// entry (i, j) = (tid / 16, tid % 16) of each thread
__device__ inline double2 cq_sum(const double2 *part, int nch, int nbp) {
  const int i = threadIdx.x / CQ, j = threadIdx.x % CQ;
  double2 t = cz(0.0, 0.0);
#pragma unroll 8
  for (int c = 0; c < nch; ++c) t = cadd(t, part[(size_t)c * CQ * CQ + threadIdx.x]);
  return i >= nbp || j >= nbp ? cz(i == j ? 1.0 : 0.0, 0.0) : t;
}

// The 16 x 16 matrices of a panel's factorisations are held in every wave alike
// (the layout of rsolve16, common.hpp), so a step needs neither LDS nor a barrier.

// Factorisations of a panel: G = R^H R (r: R, rs: the reciprocal of column c's
// diagonal entry), and with LU Q - S R = L W, S diagonal and unitary with s_j
// minus the phase of the j-th pivot (q: L below, W from the diagonal on, sr: S
// by rows, winv, yinv: 1 / w_cc and 1 / (s_c r_cc)).
struct PanelFact {
  double2 g[4], r[4], q[4], sr[4];
  double g0, rs;          // column c's diagonal entry of G; 1 / r_cc
  double2 winv, yinv;
  bool ok;                // every pivot of G above pivot_min of its column's norm
};
template <int P, bool LU>
__device__ inline void panel_fact(PanelFact &f, double pivot_min, int c, int k) {
  if constexpr (P < CQ) {
    constexpr int U = P / 4, KK = P % 4;
    const double2 grow = all_rows<KK>(f.g[U]);
    double d = row_lane<P>(grow.x);
    const bool good = d > pivot_min * row_lane<P>(f.g0);   // not with a NaN
    f.ok = f.ok && good;
    d = good ? d : 1.0;
    const double rs = rsqrt(d), rpp = d * rs;
    const double2 rp = csel(c == P, cz(rpp, 0.0), csel(c > P, cscale(grow, rs), cz(0.0, 0.0)));
    f.r[U] = csel(k == KK, rp, f.r[U]);
    f.rs = c == P ? rs : f.rs;
    const double2 gs = cscale(rp, -rs);
    // (rows and columns up to P are not read again)
#pragma unroll
    for (int u = U; u < 4; ++u) cfma(f.g[u], row_lane<P>(f.g[u]), gs);
    if constexpr (LU) {
      const double2 qrow = all_rows<KK>(f.q[U]), pv = row_lane<P>(qrow);
      const double a2 = cabs2(pv), ra = a2 > 0.0 ? rsqrt(a2) : 0.0, ab = a2 * ra;
      const double2 s = cz(a2 > 0.0 ? -pv.x * ra : -1.0, -pv.y * ra);
      const double wd = ab + rpp, wi = 1.0 / wd;   // w_PP = -s (|pv| + r_PP)
      const double2 winv = cz(-s.x * wi, s.y * wi);
      double2 w = qrow;
      cfma(w, cz(-s.x, -s.y), rp);
      const double2 mw = csel(c > P, cz(-w.x, -w.y), cz(0.0, 0.0));
#pragma unroll
      for (int u = U; u < 4; ++u) {
        const bool below = 4 * u + k > P;
        const double2 l = csel(below, cmul(row_lane<P>(f.q[u]), winv), cz(0.0, 0.0));
        cfma(f.q[u], l, mw);
        f.q[u] = csel(below && c == P, l, f.q[u]);
      }
      f.q[U] = csel(k == KK && c >= P, csel(c == P, cz(-s.x * wd, -s.y * wd), w), f.q[U]);
      f.sr[U] = csel(k == KK, s, f.sr[U]);
      f.winv = csel(c == P, winv, f.winv);
      f.yinv = csel(c == P, cz(s.x * rs, -s.y * rs), f.yinv);
    }
    panel_fact<P + 1, LU>(f, pivot_min, c, k);
  }
}

// x <- x R^{-1} for one row x (R upper in Rs, reciprocal diagonal ri), a column
// at a time taken off the later ones.  The loads of row j are tied to x[j - 1]
// (an offset of zero that the compiler cannot see through): issued all at once
// they would not fit the registers.
template <class D>
__device__ inline void cq_subst(double2 (&x)[CQ], const double2 (*Rs)[CQ + 1], const D *ri) {
  int z = 0;
#pragma unroll
  for (int j = 0; j < CQ; ++j) {
    if (j >= 2) asm volatile("" : "+v"(z) : "v"(x[j - 1].x));
    const double2 *row = &Rs[j][0] + z;
    if constexpr (sizeof(D) == sizeof(double)) x[j] = cscale(x[j], ri[j]);
    else x[j] = cmul(x[j], ri[j]);
    const double2 mx = cz(-x[j].x, -x[j].y);
#pragma unroll
    for (int i = j + 1; i < CQ; ++i) cfma(x[i], mx, row[i]);
  }
}

// side: [mat][2][16 * 16]: the top block of P R1^{-1}, then R1
__global__ __launch_bounds__(CH) void cq_solve_kernel(const MatDesc *__restrict__ descs, int k0,
                                                      const double2 *__restrict__ part, double2 *__restrict__ part2,
                                                      double2 *__restrict__ side, int nchmax, int *__restrict__ bad) {
  const MatDesc d = descs[blockIdx.y];
  const int r0 = k0 + blockIdx.x * CH, tid = threadIdx.x, r = r0 + tid;
  if (k0 >= d.n || r0 >= d.m) return;
  const int nbp = min(CQ, d.n - k0), nch = (d.m - k0 + CH - 1) / CH;
  const bool live = r < d.m;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lc = lane & 15, lk = lane >> 4;
  __shared__ double2 Gs[CQ][CQ + 1], Rs[CQ][CQ + 1];
  __shared__ double rinv[CQ];
  __shared__ double2 red[CH / 64][CQ * CQ];
  __shared__ double2 Qs[CH][CQ + 1];
  double2 x[CQ];
#pragma unroll
  for (int c = 0; c < CQ; ++c)
    x[c] = ld_or0(d.a, (size_t)(k0 + min(c, nbp - 1)) * d.lda + min(r, d.m - 1), live && c < nbp);
  Gs[tid / CQ][tid % CQ] = cq_sum(part + (size_t)blockIdx.y * nchmax * CQ * CQ, nch, nbp);
  __syncthreads();
  if (wv == 0) {
    PanelFact f;
    f.ok = true;
#pragma unroll
    for (int u = 0; u < 4; ++u) f.g[u] = Gs[4 * u + lk][lc];
    f.g0 = Gs[lc][lc].x;
    panel_fact<0, false>(f, kCholPivotMin, lc, lk);
    if (!f.ok && tid == 0) bad[blockIdx.y] = 1;
#pragma unroll
    for (int u = 0; u < 4; ++u) Rs[4 * u + lk][lc] = f.r[u];
    if (lk == 0) rinv[lc] = f.rs;
  }
  __syncthreads();
  cq_subst(x, Rs, rinv);
  double2 *sd = side + (size_t)blockIdx.y * 2 * CQ * CQ;
#pragma unroll
  for (int c = 0; c < CQ; ++c) {
    Qs[tid][c] = x[c];
    if (live && c < nbp) d.a[(size_t)(k0 + c) * d.lda + r] = x[c];
    if (blockIdx.x == 0 && tid < CQ) sd[tid * CQ + c] = x[c];
  }
  if (blockIdx.x == 0) {
    const int i = tid / CQ, j = tid % CQ;
    sd[CQ * CQ + tid] = i <= j ? Rs[i][j] : cz(0.0, 0.0);
  }
  __syncthreads();
  cq_gram([&](int row, int c) { return Qs[row][c]; }, red,
          part2 + ((size_t)blockIdx.y * nchmax + blockIdx.x) * CQ * CQ);
}

// T16: the panel's T, into its block of the matrix's T (panels of nbo columns)
// and, if tx is set, tx[mat] as well.
__global__ __launch_bounds__(CH) void cq_reflect_kernel(const MatDesc *__restrict__ descs, int k0,
                                                        const double2 *__restrict__ part2,
                                                        const double2 *__restrict__ side, int nchmax,
                                                        int *__restrict__ bad, int nbo, double2 *__restrict__ tx) {
  const MatDesc d = descs[blockIdx.y];
  // the first workgroup writes the top block and T, the others a chunk of rows each
  const int r0 = k0 + ((int)blockIdx.x - 1) * CH, tid = threadIdx.x, r = r0 + tid;
  if (k0 >= d.n || r0 >= d.m) return;
  const int nbp = min(CQ, d.n - k0), nch = (d.m - k0 + CH - 1) / CH;
  const bool below = r < d.m && r >= k0 + CQ;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, k = lane >> 4;
  __shared__ double2 Gs[CQ][CQ + 1], Rs[CQ][CQ + 1], Ws[CQ][CQ + 1];
  __shared__ double2 winv[CQ];
  double2 x[CQ];
#pragma unroll
  for (int j = 0; j < CQ; ++j)
    x[j] = ld_or0(d.a, (size_t)(k0 + min(j, nbp - 1)) * d.lda + min(r, d.m - 1), below && j < nbp);
  const double2 *sd = side + (size_t)blockIdx.y * 2 * CQ * CQ;
  PanelFact f;
  f.ok = true;
#pragma unroll
  for (int u = 0; u < 4; ++u) f.q[u] = ld_or0(sd, (4 * u + k) * CQ + c, c < nbp);   // past the last column: w = 1
  Gs[tid / CQ][tid % CQ] = cq_sum(part2 + (size_t)blockIdx.y * nchmax * CQ * CQ, nch, nbp);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) f.g[u] = Gs[4 * u + k][c];
  f.g0 = Gs[c][c].x;
  // near the identity unless the first pass failed
  panel_fact<0, true>(f, 0.1, c, k);
  if (!f.ok && blockIdx.x == 0 && tid == 0) bad[blockIdx.y] = 1;
  if (wv == 0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      Ws[4 * u + k][c] = f.q[u];
      Rs[4 * u + k][c] = f.r[u];
    }
    if (k == 0) winv[c] = f.winv;
  }
  __syncthreads();
  // the rows below: P R2^{-1} U^{-1} = P W^{-1}
  if (below) {
    cq_subst(x, Ws, winv);
#pragma unroll
    for (int j = 0; j < CQ; ++j)
      if (j < nbp) d.a[(size_t)(k0 + j) * d.lda + r] = x[j];
  }
  if (blockIdx.x > 0) return;
  if (wv == 0) {   // L
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (4 * u + k > c && c < nbp && k0 + 4 * u + k < d.m) d.a[(size_t)(k0 + c) * d.lda + k0 + 4 * u + k] = f.q[u];
  } else if (wv == 1) {   // S R2 R1
    double2 a2[4], r1[4], v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a2[u] = Rs[c][4 * u + k];
      r1[u] = sd[CQ * CQ + (4 * u + k) * CQ + c];
    }
    mul16(a2, r1, v);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (4 * u + k <= c && c < nbp) d.a[(size_t)(k0 + c) * d.lda + k0 + 4 * u + k] = cmul(f.sr[u], v[u]);
  } else if (wv == 2) {   // T = -U S^{-1} L^{-H} = -W (L^H S R2)^{-1}
    double2 lh[4], sr[4], y[4], t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int m = 4 * u + k;
      lh[u] = csel(m > c, cconj(f.q[u]), cz(m == c ? 1.0 : 0.0, 0.0));
      sr[u] = cmul(f.sr[u], f.r[u]);
      t[u] = csel(m <= c, cz(-f.q[u].x, -f.q[u].y), cz(0.0, 0.0));
    }
    mul16(lh, sr, y);
    rsolve16<0>(t, y, f.yinv, c);
    const int o = k0 % nbo;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = 4 * u + k;
      const double2 v = csel(i <= c && c < nbp, t[u], cz(0.0, 0.0));
      if (i == c && i < nbp) d.tau[k0 + i] = v;
      d.T[(size_t)(k0 / nbo) * nbo * nbo + (size_t)(o + c) * nbo + o + i] = v;
      if (tx) tx[(size_t)blockIdx.y * CQ * CQ + c * CQ + i] = v;
    }
  }
}

// Y columns: which = 0 -> trailing columns of the matrix after the panel,
// which = 1 -> columns [0, rank) of d.u, which = 2 -> columns [k0, rank) of
// d.u (forming Q from the identity: the reflectors of the panel at k0 and
// later leave columns below k0 of the identity as they are).
__device__ inline void y_source(const MatDesc &d, int k0, int nbp, int which, double2 *&B, int &ldb,
                                int &nb_cols) {
  if (which == 0) {
    nb_cols = d.n - k0 - nbp;
    // after the last panel there are no trailing columns and column k0 + nbp
    // is past the end of the matrix; masked loads (ld_or0) still read B[0],
    // so B then points at the matrix's first column instead
    B = d.a + (size_t)(nb_cols > 0 ? k0 + nbp : 0) * d.lda;
    ldb = d.lda;
  } else {
    B = d.u;
    ldb = ldu_of(d);
    nb_cols = d.rank[0];
    if (which == 2) {
      // with no columns left B stays at column 0, so that masked loads
      // (ld_or0, which read B[0]) stay inside the matrix
      const bool some = k0 < nb_cols;
      B += some ? (size_t)k0 * ldb : 0;
      nb_cols = some ? nb_cols - k0 : 0;
    }
  }
}

// Element (r, c) of Y = [V | B] (the nv = NB columns of the panel's
// Householder vectors first when withV, then the ny - nv columns of B),
// zero for rows r >= rend and columns c >= ny: one load, whose base is a
// column inside its matrix also when the element is masked (ld_or0 then
// reads the base's first element).
__device__ inline double2 yel(const MatDesc &d, int k0, int nv, const double2 *B, int ldb, int ny, int r, int c,
                              int rend) {
  const bool isv = c < nv;
  const int vc = k0 + c;   // matrix column of a V column
  const bool vin = isv && vc < d.n;
  const double2 *p = isv ? d.a + (size_t)(vin ? vc : 0) * d.lda : B + (size_t)(c < ny ? c - nv : 0) * ldb;
  const bool ok = r < rend && (isv ? (vin && r > vc) : c < ny);
  const double2 x = ld_or0(p, r, ok);
  return csel(vin && r == vc && r < rend, cz(1.0, 0.0), x);
}

// P[mat][kc][i][c] = sum over rows of slice kc of conj(V[r][i]) Y[r][c],
// Y = [V | B] (withV) or B, on the FP64 matrix cores.  The slice's rows are
// staged through LDS KS at a time (coalesced loads down the columns, the
// next stage's loads issued before the current stage's products); a 16 x 16
// tile of P is one v_mfma_f64_16x16x4f64 chain per real product (four per
// complex one), the NB x YT tile of the workgroup split over its four waves
// as VhyShape says.  cend (which = 0): the trailing columns end before
// matrix column cend.
template <int NB>
__global__ __launch_bounds__(256, VhyShape<NB>::OCC) void bqr_vhy_kernel(const MatDesc *__restrict__ descs, int k0,
                                                                        int which, int withV, int cend,
                                                                        double2 *__restrict__ P, int ldp,
                                                                        int nkcmax, int KR) {
  using S = VhyShape<NB>;
  constexpr int YT = S::YT, IB = S::IB, CB = S::CB, DB = S::DB;
  constexpr int NWI = NB / 16 / IB;   // waves along the rows of P
  static_assert(NWI * (YT / 16 / CB) == 4, "four waves cover the tile");
  const MatDesc d = descs[blockIdx.z];
  if (k0 >= d.n) return;
  const int nbp = min(NB, d.n - k0);
  double2 *B;
  int ldb, nb_cols;
  y_source(d, k0, nbp, which, B, ldb, nb_cols);
  if (which == 0) nb_cols = min(nb_cols, cend - (k0 + nbp));
  const int nv = withV ? NB : 0;
  const int ny = nv + max(nb_cols, 0);
  const int c0 = blockIdx.x * YT;
  if (c0 >= ny) return;
  const int rbeg = k0 + blockIdx.y * KR;
  if (rbeg >= d.m) return;
  const int rend = min(d.m, rbeg + KR);
  __shared__ double2 Vs[DB + 1][KS][NB + 1];
  __shared__ double2 Ys[DB + 1][KS][YT + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int l16 = lane & 15, k4 = lane >> 4;
  const int wi = wv % NWI, wc = wv / NWI;
  dx4 re[IB][CB], im[IB][CB];
#pragma unroll
  for (int u = 0; u < IB; ++u)
#pragma unroll
    for (int v = 0; v < CB; ++v) {
      re[u][v] = dx4{0.0, 0.0, 0.0, 0.0};
      im[u][v] = re[u][v];
    }
  double2 vv[KS * NB / 256], yy[KS * YT / 256];
  auto load_stage = [&](int r0) {
#pragma unroll
    for (int u = 0; u < KS * NB / 256; ++u) {
      const int idx = tid + 256 * u, rr = idx % KS, i = idx / KS;
      const int r = r0 + rr;
      vv[u] = csel(r < rend, vel(d, k0, i, r), cz(0.0, 0.0));
    }
#pragma unroll
    for (int u = 0; u < KS * YT / 256; ++u) {
      const int idx = tid + 256 * u, rr = idx % KS, cc = idx / KS;
      yy[u] = yel(d, k0, nv, B, ldb, ny, r0 + rr, c0 + cc, rend);
    }
  };
  auto store_stage = [&](int buf) {
#pragma unroll
    for (int u = 0; u < KS * NB / 256; ++u) {
      const int idx = tid + 256 * u;
      Vs[buf][idx % KS][idx / KS] = vv[u];
    }
#pragma unroll
    for (int u = 0; u < KS * YT / 256; ++u) {
      const int idx = tid + 256 * u;
      Ys[buf][idx % KS][idx / KS] = yy[u];
    }
  };
  auto products = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < KS; kk += 4) {
      // A[i][k] = conj(V[row k][col i]) (lane l16 + 16 k4 holds A[l16][k4]),
      // B[k][c] = Y[row k][col c]
      double2 a[IB], y[CB];
#pragma unroll
      for (int u = 0; u < IB; ++u) a[u] = Vs[buf][kk + k4][16 * (wi * IB + u) + l16];
#pragma unroll
      for (int v = 0; v < CB; ++v) y[v] = Ys[buf][kk + k4][16 * (wc * CB + v) + l16];
#pragma unroll
      for (int u = 0; u < IB; ++u)
#pragma unroll
        for (int v = 0; v < CB; ++v) {
          re[u][v] = mfma_f64(a[u].x, y[v].x, re[u][v]);
          re[u][v] = mfma_f64(a[u].y, y[v].y, re[u][v]);
          im[u][v] = mfma_f64(a[u].x, y[v].y, im[u][v]);
          im[u][v] = mfma_f64(-a[u].y, y[v].x, im[u][v]);
        }
    }
  };
  load_stage(rbeg);
  if (DB) {
    int buf = 0;
    store_stage(0);
    __syncthreads();
    for (int r0 = rbeg; r0 < rend; r0 += KS) {
      const bool more = r0 + KS < rend;
      if (more) load_stage(r0 + KS);
      products(buf);
      if (more) store_stage(buf ^ 1);   // the other buffer: read by no wave since the last barrier
      __syncthreads();
      buf ^= 1;
    }
  } else {
    for (int r0 = rbeg; r0 < rend; r0 += KS) {
      store_stage(0);
      __syncthreads();
      if (r0 + KS < rend) load_stage(r0 + KS);
      products(0);
      __syncthreads();
    }
  }
  // lane l16 + 16 k4 holds P[16 (wi IB + u) + k4 + 4 e][column block's l16] in element e
  double2 *out = P + ((size_t)blockIdx.z * nkcmax + blockIdx.y) * NB * ldp;
#pragma unroll
  for (int v = 0; v < CB; ++v) {
    const int c = c0 + 16 * (wc * CB + v) + l16;
    if (c < ny) {
#pragma unroll
      for (int u = 0; u < IB; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          out[(size_t)(16 * (wi * IB + u) + k4 + 4 * e) * ldp + c] = cz(re[u][v][e], im[u][v][e]);
    }
  }
}

// T of the panel (forward, columnwise): H_0 ... H_{NB-1} = I - V T V^H.
// Diagonal blocks of 16 by the column recurrence T[i][i] = tau_i,
// T[0:i, i] = -tau_i T[0:i, 0:i] (V^H V)[0:i, i], one wave a block, the
// blocks side by side (16 steps for any NB); then adjacent blocks of h = 16, 32
// joined as T12 = -T1 (V1^H V2) T2 (the product of two block reflectors).
// V^H V from the slices of P.  Written to the matrix's T of panel k0 / NB,
// or to Tx[mat] if Tx is set (an inner panel's T, needed only until its
// update is done).
// threads of the T kernel: the sum over the slices is spread over all of them
// (64-column panels over 25 slices: 94 us with 256)
template <int NB> struct TThreads { static constexpr int N = NB * NB / 4 < 256 ? 256 : NB * NB / 4; };
template <int NB>
__global__ __launch_bounds__(TThreads<NB>::N) void bqr_t_kernel(const MatDesc *__restrict__ descs, int k0,
                                                    const double2 *__restrict__ P, int ldp, int nkcmax,
                                                    double2 *__restrict__ Tx, int KR, int diag) {
  constexpr int TT = TThreads<NB>::N;
  static_assert(NB % 16 == 0 && NB <= 64, "diagonal blocks of 16, one wave each");
  const MatDesc d = descs[blockIdx.x];
  if (k0 >= d.n) return;
  const int nbp = min(NB, d.n - k0);
  const int nkc = (d.m - k0 + KR - 1) / KR;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ double2 gram[NB][NB + 1];
  __shared__ double2 Tsh[NB][NB + 1];
  __shared__ double2 X[NB / 2][NB / 2 + 1];
  const double2 *base = P + (size_t)blockIdx.x * nkcmax * NB * ldp;
  {
    // strict upper part, summed over the slices (consecutive threads along a row of P)
    double2 t[NB * NB / TT];
#pragma unroll
    for (int u = 0; u < NB * NB / TT; ++u) t[u] = cz(0.0, 0.0);
#pragma unroll 4
    for (int kc = 0; kc < nkc; ++kc) {
#pragma unroll
      for (int u = 0; u < NB * NB / TT; ++u) {
        const int idx = tid + TT * u, i = idx % NB, g = idx / NB;
        t[u] = cadd(t[u], ld_or0(base, ((size_t)kc * NB + g) * ldp + i, diag ? g / 16 < i / 16 && i < nbp : g < i && i < nbp));
      }
    }
#pragma unroll
    for (int u = 0; u < NB * NB / TT; ++u) {
      const int idx = tid + TT * u;
      gram[idx / NB][idx % NB] = t[u];
    }
    for (int idx = tid; idx < NB * (NB + 1); idx += TT) Tsh[idx / (NB + 1)][idx % (NB + 1)] = cz(0.0, 0.0);
  }
  __syncthreads();
  // diagonal blocks, all at once: wave w < NB / 16 takes block w (lane l: row 16 w + l)
  __shared__ double2 tmp[NB];
  const bool blk = wv < NB / 16 && lane < 16;
  const int o = 16 * wv;
  if (diag) {   // given (cq_reflect_kernel, bqr_panel_kernel)
    const double2 *T = d.T + (size_t)(k0 / NB) * NB * NB;
    for (int idx = tid; idx < NB * NB; idx += TT) {
      const int r = idx % NB, c = idx / NB;
      if (r / 16 == c / 16 && r <= c && c < nbp) Tsh[r][c] = T[idx];
    }
    __syncthreads();
  }
  for (int i = 0; i < 16 && !diag; ++i) {
    const int ci = o + i;
    const double2 ti = blk && ci < nbp ? d.tau[k0 + ci] : cz(0.0, 0.0);
    if (blk && lane < i) tmp[o + lane] = cmul(cz(-ti.x, -ti.y), gram[o + lane][ci]);
    __syncthreads();
    if (blk && lane < i) {
      double2 acc = cz(0.0, 0.0);
      for (int g = lane; g < i; ++g) cfma(acc, Tsh[o + lane][o + g], tmp[o + g]);
      Tsh[o + lane][ci] = acc;
    }
    if (blk && lane == i) Tsh[ci][ci] = ti;
    __syncthreads();
  }
  for (int h = 16; h < NB; h *= 2) {
    // pairs (o, o + h), o = 2 h p: X = G12 T2, then T12 = -T1 X
    const int npair = NB / (2 * h), nout = npair * h * h;
    for (int idx = tid; idx < nout; idx += TT) {
      const int p = idx / (h * h), r = (idx / h) % h, c = idx % h, o = 2 * h * p;
      double2 acc = cz(0.0, 0.0);
      for (int g = 0; g <= c; ++g) cfma(acc, gram[o + r][o + h + g], Tsh[o + h + g][o + h + c]);
      X[p * h + r][c] = acc;
    }
    __syncthreads();
    for (int idx = tid; idx < nout; idx += TT) {
      const int p = idx / (h * h), r = (idx / h) % h, c = idx % h, o = 2 * h * p;
      double2 acc = cz(0.0, 0.0);
      for (int g = r; g < h; ++g) cfma(acc, Tsh[o + r][o + g], X[p * h + g][c]);
      Tsh[o + r][o + h + c] = cz(-acc.x, -acc.y);
    }
    __syncthreads();
  }
  double2 *T = Tx ? Tx + (size_t)blockIdx.x * NB * NB : d.T + (size_t)(k0 / NB) * NB * NB;
  for (int idx = tid; idx < NB * NB; idx += TT) {
    const int r = idx % NB, c = idx / NB;
    T[idx] = (r <= c && c < nbp) ? Tsh[r][c] : cz(0.0, 0.0);
  }
}

// W2[mat][i][c] = sum_h op(T)[i][h] W[h][c], W = V^H B summed over the slices;
// op(T) = T^H (trans, QR) or T; T from Tx[mat] if Tx is set (bqr_t_kernel).
// T is upper triangular: a workgroup stages its triangle once in LDS (packed
// by columns, entry (r, c) at c (c + 1) / 2 + r, half of the square's LDS, so
// three workgroups share a CU) and then takes W2T-column tiles gridDim.x
// apart, so that a batch of many small matrices stages each T once per
// several tiles instead of once per tile.  A thread holds one column of the
// tile and the NB / 16 rows g, g + 16, ... and accumulates them side by side.
// (256-obstacle batch, 64-column panels: 1.65 ms a launch with the square T
// staged per 16-column tile at one workgroup a CU and one output at a time.)
template <int NB>
__global__ __launch_bounds__(256, 3) void bqr_w2_kernel(const MatDesc *__restrict__ descs, int k0, int which,
                                                     int withV, int trans, int cend,
                                                     const double2 *__restrict__ P, int ldp, int nkcmax,
                                                     double2 *__restrict__ W2, int ldw,
                                                     const double2 *__restrict__ Tx, int KR) {
  static_assert(W2T == 16 && NB % 16 == 0, "a thread: one column of the tile, rows 16 apart");
  constexpr int R = NB / 16;
  const MatDesc d = descs[blockIdx.y];
  if (k0 >= d.n) return;
  const int nbp = min(NB, d.n - k0);
  double2 *B;
  int ldb, nb_cols;
  y_source(d, k0, nbp, which, B, ldb, nb_cols);
  if (which == 0) nb_cols = min(nb_cols, cend - (k0 + nbp));
  if ((int)blockIdx.x * W2T >= nb_cols) return;
  const int nv = withV ? NB : 0;
  const int nkc = (d.m - k0 + KR - 1) / KR;
  __shared__ double2 Tp[NB * (NB + 1) / 2];
  __shared__ double2 Ws[NB][W2T + 1];
  const int tid = threadIdx.x, cc = tid % W2T, g = tid / W2T;
  const double2 *T = Tx ? Tx + (size_t)blockIdx.y * NB * NB : d.T + (size_t)(k0 / NB) * NB * NB;
  for (int idx = tid; idx < NB * NB; idx += 256) {
    const int r = idx % NB, c = idx / NB;
    if (r <= c) Tp[c * (c + 1) / 2 + r] = T[idx];
  }
  const double2 *base = P + (size_t)blockIdx.y * nkcmax * NB * ldp;
  double2 *out = W2 + (size_t)blockIdx.y * NB * ldw;
  for (int c0 = blockIdx.x * W2T; c0 < nb_cols; c0 += gridDim.x * W2T) {
    const int c = c0 + cc;
    const bool live = c < nb_cols;
    double2 t[R];
#pragma unroll
    for (int u = 0; u < R; ++u) t[u] = cz(0.0, 0.0);
#pragma unroll 6
    for (int kc = 0; kc < nkc; ++kc) {
#pragma unroll
      for (int u = 0; u < R; ++u)
        t[u] = cadd(t[u], ld_or0(base, ((size_t)kc * NB + g + 16 * u) * ldp + nv + c, live));
    }
    __syncthreads();   // Tp staged; the previous tile's products are done with Ws
#pragma unroll
    for (int u = 0; u < R; ++u) Ws[g + 16 * u][cc] = t[u];
    __syncthreads();
    double2 acc[R];
#pragma unroll
    for (int u = 0; u < R; ++u) acc[u] = cz(0.0, 0.0);
    if (trans) {
#pragma unroll 4
      for (int h = 0; h < NB; ++h) {
        const double2 w = Ws[h][cc];
#pragma unroll
        for (int u = 0; u < R; ++u) {
          const int i = g + 16 * u;
          if (h <= i) cfmac(acc[u], Tp[i * (i + 1) / 2 + h], w);
        }
      }
    } else {
#pragma unroll 4
      for (int h = 0; h < NB; ++h) {
        const double2 w = Ws[h][cc];
#pragma unroll
        for (int u = 0; u < R; ++u) {
          const int i = g + 16 * u;
          if (h >= i) cfma(acc[u], Tp[h * (h + 1) / 2 + i], w);
        }
      }
    }
    if (live) {
#pragma unroll
      for (int u = 0; u < R; ++u) out[(size_t)(g + 16 * u) * ldw + c] = acc[u];
    }
  }
}

// C -= V W2 on the FP64 matrix cores, in transposed orientation (D = W2^T
// V^T, so that a lane's outputs run down a column: 256-byte stores).  A wave
// updates 2 x 2 tiles of 16 x 16 (32 rows x 32 columns), each a real and an
// imaginary accumulator, and loads the next k-step's fragments of W2 and V
// while it multiplies the current ones; the four waves of a workgroup stack
// along the rows (128 x 32), three workgroups a CU.  (Measured on 8 matrices
// 4608 x 1275 with 64-column panels: 51 TFLOP/s, against 40 for 32 x 64
// wave tiles at two waves a SIMD and 26 for one 16-column block a wave.)
// cend (which = 0): the trailing columns end before matrix column cend.
struct UpdShape {
  static constexpr int RB = 2;              // 16-row blocks a wave
  static constexpr int CB = 2;              // 16-column blocks a wave
  static constexpr int UR = 4 * 16 * RB;    // rows of a workgroup tile (waves along the rows)
  static constexpr int UC = 16 * CB;        // columns of a workgroup tile
};

template <int NB>
__global__ __launch_bounds__(256, 3) void bqr_update_kernel(const MatDesc *__restrict__ descs, int k0, int which,
                                                            int cend, const double2 *__restrict__ W2, int ldw) {
  using S = UpdShape;
  constexpr int RB = S::RB, CB = S::CB;
  const MatDesc d = descs[blockIdx.z];
  if (k0 >= d.n) return;
  const int nbp = min(NB, d.n - k0);
  double2 *B;
  int ldb, nb_cols;
  y_source(d, k0, nbp, which, B, ldb, nb_cols);
  if (which == 0) nb_cols = min(nb_cols, cend - (k0 + nbp));
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int l16 = lane & 15, k4 = lane >> 4;
  // this wave's first row and column (no barriers: an idle wave may leave)
  const int rw = k0 + blockIdx.y * S::UR + wv * 16 * RB;
  const int cw = blockIdx.x * S::UC;
  if (rw >= d.m || cw >= nb_cols) return;
  const int ncb = min(CB, (nb_cols - cw + 15) / 16);   // column blocks holding columns (wave-uniform)
  const int nrb = min(RB, (d.m - rw + 15) / 16);       // row blocks holding rows
  const double2 *w2 = W2 + (size_t)blockIdx.z * NB * ldw;
  dx4 re[RB][CB], im[RB][CB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      re[rb][cb] = dx4{0.0, 0.0, 0.0, 0.0};
      im[rb][cb] = re[rb][cb];
    }
  // A[c][i] = W2[i][c] (lane l16 + 16 k4 holds A[l16][k4]); B[i][r] = V[r][i]
  auto load = [&](int ks, double2 (&a)[CB], double2 (&v)[RB]) {
    const int i = 4 * ks + k4;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int c = cw + 16 * cb + l16;
      a[cb] = ld_or0(w2, (size_t)i * ldw + c, c < nb_cols);
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) v[rb] = vel(d, k0, i, rw + 16 * rb + l16);   // zero for rows >= m
  };
  auto mma = [&](const double2 (&a)[CB], const double2 (&v)[RB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        if (rb >= nrb || cb >= ncb) continue;   // wave-uniform: a block with no rows or no columns
        re[rb][cb] = mfma_f64(a[cb].x, v[rb].x, re[rb][cb]);
        re[rb][cb] = mfma_f64(-a[cb].y, v[rb].y, re[rb][cb]);
        im[rb][cb] = mfma_f64(a[cb].x, v[rb].y, im[rb][cb]);
        im[rb][cb] = mfma_f64(a[cb].y, v[rb].x, im[rb][cb]);
      }
  };
  static_assert(NB % 8 == 0, "k-steps in pairs");
  double2 a0[CB], v0[RB], a1[CB], v1[RB];
  load(0, a0, v0);
#pragma unroll
  for (int ks = 0; ks < NB / 4; ks += 2) {
    load(ks + 1, a1, v1);
    mma(a0, v0);
    if (ks + 2 < NB / 4) load(ks + 2, a0, v0);
    mma(a1, v1);
  }
  // lane l16 + 16 k4 holds D[k4 + 4 e][l16] in element e of tile (rb, cb):
  // column cw + 16 cb + k4 + 4 e, row rw + 16 rb + l16
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = cw + 16 * cb + k4 + 4 * e;
      if (c >= nb_cols) continue;
      double2 *col = B + (size_t)c * ldb;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int r = rw + 16 * rb + l16;
        if (r < d.m) {
          const double2 x = col[r];
          col[r] = cz(x.x - re[rb][cb][e], x.y - im[rb][cb][e]);
        }
      }
    }
}

// Rows of a V^H Y slice for `rows` rows and ny columns of Y: VhyShape's or shorter,
// down to 64, by what a launch takes.  A compute unit with one workgroup needs
// 1.3 of a workgroup's share of one that is full, with q of them q; a slice has a
// cost of 40 rows, and another slice costs W2 and T that add it 3 rows.  4
// matrices of 4096 x 1472, 46 launches with 24 to 736 workgroups of 512 rows:
// 7.2 -> 5.9 ms, W2 and T 1.5 -> 1.8 (one choice for a whole factorisation by its
// average panel before).
int vhy_slice_rows(int nb, int nmat, int rows, int ny) {
  int best = nb == 64 ? VhyShape<64>::KR : (nb == 32 ? VhyShape<32>::KR : VhyShape<16>::KR);
  double cost = 0.0;
  for (int kr = best; kr >= KRMIN; kr /= 2) {
    const int nkc = cdiv(std::max(rows, 1), kr);
    const long q = ((long)cdiv(std::max(ny, 1), 64) * nkc * nmat + 255) / 256;
    if (q > 4 && cost == 0.0) break;   // full as it is
    const double c = (q <= 1 ? 1.3 : (double)q) * (kr + 40) + 3.0 * nkc;
    if (cost == 0.0 || c < cost) {
      cost = c;
      best = kr;
    }
  }
  return best;
}

struct ApplyWork {
  DevBuf P, W2;
  int ldw = 0;
  // P for the panels of a factorisation of ncols columns or an application to
  // them (apply_panel enlarges it for a panel that needs more)
  void size(int nmat, int mmax, int ncols, int nb) {
    ldw = std::max(ncols, 1);
    size_t most = 0;
    for (int k0 = 0; k0 == 0 || k0 < ncols; k0 += nb) {
      const int ny = nb + ncols - k0;
      most = std::max(most, (size_t)cdiv(std::max(mmax - k0, 1), vhy_slice_rows(nb, nmat, mmax - k0, ny)) * ny);
    }
    P.alloc((size_t)nmat * most * nb * sizeof(double2));
    W2.alloc((size_t)nmat * nb * ldw * sizeof(double2));
  }
};

// C <- (I - V T V^H)^{op} C for the panel at k0 (which/withV/trans as above).
// cend: with which = 0, the trailing columns end before matrix column cend;
// Tx: T of the panel to and from Tx[mat] instead of the matrix's T.
constexpr int kNoEnd = 0x7fffffff;
template <int NB>
void apply_panel(const MatDesc *descs, int nmat, int mmax, int ncols_max, int k0, int which, int withV,
                 int trans, ApplyWork &w, bool build_t, hipStream_t s, int cend = kNoEnd,
                 double2 *Tx = nullptr, int diag = 0) {
  const int ny = (withV ? NB : 0) + ncols_max;
  const int kr = vhy_slice_rows(NB, nmat, mmax - k0, ny), nkc = cdiv(std::max(mmax - k0, 1), kr);
  const size_t need = (size_t)nmat * nkc * NB * ny * sizeof(double2);
  if (w.P.bytes < need) w.P.alloc(need);
  if (ny > 0)
    hipLaunchKernelGGL(bqr_vhy_kernel<NB>, dim3(cdiv(ny, VhyShape<NB>::YT), nkc, nmat), dim3(256), 0, s, descs, k0, which, withV,
                       cend, w.P.as<double2>(), ny, nkc, kr);
  if (build_t)
    hipLaunchKernelGGL(bqr_t_kernel<NB>, dim3(nmat), dim3(TThreads<NB>::N), 0, s, descs, k0, w.P.as<double2>(), ny, nkc,
                       Tx, kr, diag);
  if (ncols_max > 0) {
    const int w2x = std::min(cdiv(ncols_max, W2T), std::max(1, cdiv(W2WG, nmat)));
    hipLaunchKernelGGL(bqr_w2_kernel<NB>, dim3(w2x, nmat), dim3(256), 0, s, descs, k0, which,
                       withV, trans, cend, w.P.as<double2>(), ny, nkc, w.W2.as<double2>(), w.ldw, Tx, kr);
    hipLaunchKernelGGL(bqr_update_kernel<NB>,
                       dim3(cdiv(ncols_max, UpdShape::UC), cdiv(std::max(mmax - k0, 1), UpdShape::UR), nmat),
                       dim3(256), 0, s, descs, k0, which, cend, w.W2.as<double2>(), w.ldw);
  }
  HIP_CHECK(hipGetLastError());
}

// Householder vectors and tau of the columns [k0, k0 + NI) (NI = 16), the
// column steps of bqr_col_kernel or the one-launch bqr_panel_kernel
struct PanelWork {
  static constexpr int NI = PNB;
  DevBuf part, side;
  int nchmax = 0;
  int *bad = nullptr;   // given: Cholesky panels, [nmat] flags of matrices they could not factor
  void size(int nmat, int mmax, int *flags) {
    nchmax = cdiv(mmax, CH);
    bad = flags;
    const int np = bad ? CQ * CQ : NI + 1, ns = bad ? CQ * CQ : NI;
    part.alloc((size_t)nmat * 2 * nchmax * np * sizeof(double2));
    side.alloc((size_t)nmat * 2 * ns * sizeof(double2));
  }
  // whether factor() brings T of the panel at k0
  bool brings_t(int mmax, int k0) const { return bad || mmax - k0 <= PTMAX; }
  void factor(const MatDesc *descs, int nmat, int mmax, int nmax, int k0, hipStream_t s, int nbo, double2 *tx) {
    const int nbp = std::min(NI, nmax - k0);
    if (bad) {
      const dim3 g(cdiv(std::max(mmax - k0, 1), CH), nmat);
      double2 *p2 = part.as<double2>() + (size_t)nmat * nchmax * CQ * CQ;
      hipLaunchKernelGGL(cq_gram_kernel, g, dim3(CH), 0, s, descs, k0, part.as<double2>(), nchmax);
      hipLaunchKernelGGL(cq_solve_kernel, g, dim3(CH), 0, s, descs, k0, part.as<double2>(), p2, side.as<double2>(),
                         nchmax, bad);
      hipLaunchKernelGGL(cq_reflect_kernel, dim3(g.x + 1, g.y), dim3(CH), 0, s, descs, k0, p2, side.as<double2>(), nchmax, bad,
                         nbo, tx);
    } else if (mmax - k0 <= PTMAX) {
      // every matrix's remaining rows fit one workgroup: the panel in one launch,
      // with the fewest rows a thread that eight waves can take (a step of four
      // rows a thread 1.2 us, of eight 1.8, of sixteen 2.5 to 3.4)
      const int rows = std::max(mmax - k0, 1);
      if (rows <= 128)
        hipLaunchKernelGGL((bqr_panel_kernel<4, 8>), dim3(nmat), dim3(64 * cdiv(rows, 16)), 0, s, descs, k0, nbo, tx);
      else if (rows <= 256)
        hipLaunchKernelGGL((bqr_panel_kernel<8, 8>), dim3(nmat), dim3(64 * cdiv(rows, 32)), 0, s, descs, k0, nbo, tx);
      else
        hipLaunchKernelGGL((bqr_panel_kernel<16, 16>), dim3(nmat), dim3(64 * cdiv(rows, 64)), 0, s, descs, k0, nbo,
                           tx);
    } else {
      const int nch = cdiv(std::max(mmax - k0, 1), CH);
      for (int st = -1; st < nbp; ++st)
        hipLaunchKernelGGL(bqr_col_kernel<NI>, dim3(nch, nmat), dim3(CH), 0, s, descs, k0, st,
                           part.as<double2>(), side.as<double2>(), nchmax);
    }
    HIP_CHECK(hipGetLastError());
  }
};

// Two-level blocking: panels of NB columns (the block reflector whose T the
// matrix keeps and whose trailing update is one pass over the matrix)
// factored as NB / 16 inner panels of 16 columns, each applied only to the
// rest of its NB-column panel (its T in a scratch buffer).  NB = 16 is the
// plain one-level form.  One panel at a time (panel(K0)), so that a caller
// may act between panels (the sketched pivoted QR moves columns).
template <int NB>
struct BlockedQR {
  static constexpr int NI = PanelWork::NI;
  static_assert(NB % NI == 0, "outer panels are whole inner panels");
  const MatDesc *descs = nullptr;
  int nmat = 0, nmax = 0, mmax = 0;
  PanelWork pw;
  ApplyWork w, wi;
  DevBuf tx;
  BlockedQR(const MatDesc *d, const std::vector<MatDesc> &h, int *bad = nullptr) : descs(d), nmat((int)h.size()) {
    for (const auto &m : h) {
      nmax = std::max(nmax, m.n);
      mmax = std::max(mmax, m.m);
    }
    if (nmax == 0 || nmat == 0) return;
    pw.size(nmat, mmax, bad);
    w.size(nmat, mmax, nmax, NB);
    if (NB > NI) {
      wi.size(nmat, mmax, NB - NI, NI);
      tx.alloc((size_t)nmat * NI * NI * sizeof(double2));
    }
  }
  // the panel of columns [K0, K0 + NB) and its update of the columns after it
  void panel(int K0, hipStream_t s) {
    // Cholesky and one-launch panels bring their T: the inner applies need no V^H V
    for (int k0 = K0; k0 < std::min(K0 + NB, nmax); k0 += NI) {
      pw.factor(descs, nmat, mmax, nmax, k0, s, NB, NB > NI ? tx.as<double2>() : nullptr);
      const int rest = std::min(K0 + NB, nmax) - (k0 + NI);   // inner columns still to update
      const bool given = pw.brings_t(mmax, k0);
      if (NB > NI && rest > 0)
        apply_panel<NI>(descs, nmat, mmax, rest, k0, 0, !given, 1, wi, !given, s, K0 + NB, tx.as<double2>());
    }
    const bool given = pw.brings_t(mmax, K0);   // then also of the panels after it
    const bool whole = NB == NI && given;   // T complete
    apply_panel<NB>(descs, nmat, mmax, std::max(0, nmax - K0 - NB), K0, 0, !whole, 1, w, !whole, s, kNoEnd, nullptr,
                    given);
  }
};

template <int NB>
void qr_factor_t(const MatDesc *descs, const std::vector<MatDesc> &h, hipStream_t s, int *bad) {
  BlockedQR<NB> q(descs, h, bad);
  for (int K0 = 0; K0 < q.nmax; K0 += NB) q.panel(K0, s);
}

template <int NB>
void qr_form_u_t(const MatDesc *descs, const std::vector<MatDesc> &h, int maxrank, hipStream_t s,
                 bool from_identity) {
  int nmax = 0, mmax = 0;
  for (const auto &d : h) {
    nmax = std::max(nmax, d.n);
    mmax = std::max(mmax, d.m);
  }
  const int nmat = (int)h.size();
  if (maxrank <= 0 || nmax == 0) return;
  ApplyWork w;
  w.size(nmat, mmax, maxrank, NB);
  for (int k0 = ((nmax - 1) / NB) * NB; k0 >= 0; k0 -= NB) {
    if (from_identity)
      apply_panel<NB>(descs, nmat, mmax, std::max(0, maxrank - k0), k0, 2, 0, 0, w, false, s);
    else
      apply_panel<NB>(descs, nmat, mmax, maxrank, k0, 1, 0, 0, w, false, s);
  }
}

}  // namespace

// ------------------------------------------------------- panel width tuner
// The panel width trades the panel's column steps (one reduction over all
// rows per column, whatever the width) against the passes of the trailing
// update over the matrix (one per panel): which wins depends on the
// matrices' shape and the GPU.  The first batch of a size class (the number
// of rows and of columns, each rounded to a half octave) on a GPU model
// times the QR of up to 8 of its matrices with every width, followed by the
// formation of U from the identity that every caller does next (64-wide
// reflectors: a narrower QR leaves their T to be rebuilt), and keeps the
// fastest; later batches of that class reuse it.  MFS_QR_NB = 16, 32 or 64
// fixes the width; MFS_QR_TUNE_FILE names a file that keeps the choices
// across processes (one "key width" line per class).
namespace {

// U = the first n columns of the identity (the tuner's U formation)
__global__ void tune_identity_kernel(const MatDesc *__restrict__ descs) {
  const MatDesc d = descs[blockIdx.y];
  const int c = blockIdx.x;
  if (c >= d.n) return;
  for (int r = threadIdx.x; r < d.m; r += blockDim.x) d.u[(size_t)c * d.ldu + r] = cz(r == c ? 1.0 : 0.0, 0.0);
}

std::mutex g_tune_mu;
std::map<std::string, int> g_tune;
bool g_tune_loaded = false;

int half_octave(int x) { return x <= 1 ? 0 : (int)std::floor(2.0 * std::log2((double)x)); }

std::string tune_key(int mmax, int nmax) {
  int dev = 0;
  HIP_CHECK(hipGetDevice(&dev));
  hipDeviceProp_t prop;
  HIP_CHECK(hipGetDeviceProperties(&prop, dev));
  std::string arch = prop.gcnArchName;
  const size_t colon = arch.find(':');
  if (colon != std::string::npos) arch = arch.substr(0, colon);
  return arch + "/m" + std::to_string(half_octave(mmax)) + "/n" + std::to_string(half_octave(nmax));
}

void tune_load() {   // g_tune_mu held
  if (g_tune_loaded) return;
  g_tune_loaded = true;
  const char *f = std::getenv("MFS_QR_TUNE_FILE");
  if (!f) return;
  std::FILE *fp = std::fopen(f, "r");
  if (!fp) return;
  char key[256];
  int nb = 0;
  while (std::fscanf(fp, "%255s %d", key, &nb) == 2)
    if (nb == 16 || nb == 32 || nb == 64) g_tune[key] = nb;
  std::fclose(fp);
}

void tune_store(const std::string &key, int nb) {   // g_tune_mu held
  g_tune[key] = nb;
  if (const char *f = std::getenv("MFS_QR_TUNE_FILE")) {
    if (std::FILE *fp = std::fopen(f, "a")) {
      std::fprintf(fp, "%s %d\n", key.c_str(), nb);
      std::fclose(fp);
    }
  }
}

}  // namespace

void qr_form_u(const MatDesc *descs, const std::vector<MatDesc> &h, int maxrank, hipStream_t s,
               bool from_identity, int nb);

int qr_tuned_nb(const std::vector<MatDesc> &h, hipStream_t s, bool chol) {
  if (const char *e = std::getenv("MFS_QR_NB")) {
    const int nb = std::atoi(e);
    MFS_REQUIRE(nb == 16 || nb == 32 || nb == 64, "MFS_QR_NB must be 16, 32 or 64");
    return nb;
  }
  int nmax = 0, mmax = 0;
  for (const auto &d : h) {
    nmax = std::max(nmax, d.n);
    mmax = std::max(mmax, d.m);
  }
  if (h.empty() || nmax == 0) return kQRNB;
  const std::string key = tune_key(mmax, nmax) + (chol ? "/c" : "");
  std::lock_guard<std::mutex> lk(g_tune_mu);
  tune_load();
  auto it = g_tune.find(key);
  if (it != g_tune.end()) return it->second;
  // the batch's largest matrices, copied (the QR works in place): up to 8,
  // and no more than 2^25 elements in all once the first is taken
  std::vector<int> idx(h.size());
  for (size_t i = 0; i < h.size(); ++i) idx[i] = (int)i;
  std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) {
    return (double)h[x].m * h[x].n > (double)h[y].m * h[y].n;
  });
  {
    size_t keep = 0, elems = 0;
    while (keep < idx.size() && keep < 8) {
      const size_t e = (size_t)h[idx[keep]].lda * h[idx[keep]].n;
      if (keep > 0 && elems + e > ((size_t)1 << 25)) break;
      elems += e;
      ++keep;
    }
    idx.resize(keep);
  }
  // a sample matrix of more than 2^25 elements (one matrix only) is timed on
  // its leading block of about 2^25 elements, same aspect ratio
  std::vector<int> sm(idx.size()), sn(idx.size()), sld(idx.size());
  for (size_t k = 0; k < idx.size(); ++k) {
    const MatDesc &d = h[idx[k]];
    const double f = std::min(1.0, std::sqrt((double)((size_t)1 << 25) / ((double)d.m * d.n)));
    sn[k] = std::max(1, std::min(d.n, (int)(d.n * f)));
    sm[k] = std::max(sn[k], std::min(d.m, (int)(d.m * f)));
    sld[k] = f < 1.0 ? round_up(sm[k], 16) : d.lda;
  }
  const int snmax = *std::max_element(sn.begin(), sn.end());
  std::vector<MatDesc> hc;
  std::vector<size_t> off;
  size_t tot = 0;
  for (size_t k = 0; k < idx.size(); ++k) {
    off.push_back(tot);
    // a, tau, T for the widest panel (cdiv(n, 16) panels of 64 x 64 bound
    // every width), and U (lda x n) formed from the identity
    tot += ((size_t)2 * sld[k] * sn[k] + sn[k] + (size_t)cdiv(sn[k], 16) * 64 * 64 + 16) * sizeof(double2);
  }
  DevBuf buf(tot), dd;
  for (size_t k = 0; k < idx.size(); ++k) {
    MatDesc c{};
    double2 *p = reinterpret_cast<double2 *>(static_cast<char *>(buf.p) + off[k]);
    c.a = p; c.m = sm[k]; c.n = sn[k]; c.lda = sld[k];
    c.tau = p + (size_t)c.lda * c.n;
    c.T = c.tau + c.n;
    c.u = c.T + (size_t)cdiv(c.n, 16) * 64 * 64;
    c.ldu = c.lda;
    hc.push_back(c);
  }
  DevBuf ranks(hc.size() * sizeof(int)), bad(hc.size() * sizeof(int));
  {
    std::vector<int> rk(hc.size());
    for (size_t k = 0; k < hc.size(); ++k) {
      rk[k] = hc[k].n;
      hc[k].rank = ranks.as<int>() + k;
    }
    HIP_CHECK(hipMemcpyAsync(ranks.p, rk.data(), rk.size() * sizeof(int), hipMemcpyHostToDevice, s));
    HIP_CHECK(hipStreamSynchronize(s));   // rk goes out of scope
  }
  dd.alloc(hc.size() * sizeof(MatDesc));
  HIP_CHECK(hipMemcpyAsync(dd.p, hc.data(), hc.size() * sizeof(MatDesc), hipMemcpyHostToDevice, s));
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  int best = kQRNB;
  float best_ms = 0.f;
  std::string report;
  for (int nb : {16, 32, 64}) {
    float ms = 0.f;
    // the first run loads the kernels; it is repeated unless it ran long
    // enough (50 ms) for the load to be lost in it
    for (int rep = 0; rep < 2 && (rep == 0 || ms < 50.f); ++rep) {
      for (size_t k = 0; k < idx.size(); ++k)
        HIP_CHECK(hipMemcpy2DAsync(hc[k].a, (size_t)hc[k].lda * sizeof(double2), h[idx[k]].a,
                                   (size_t)h[idx[k]].lda * sizeof(double2), (size_t)hc[k].m * sizeof(double2),
                                   hc[k].n, hipMemcpyDeviceToDevice, s));
      hipLaunchKernelGGL(tune_identity_kernel, dim3(snmax, (int)hc.size()), dim3(256), 0, s, dd.as<MatDesc>());
      HIP_CHECK(hipEventRecord(e0, s));
      qr_factor(dd.as<MatDesc>(), hc, s, nb, chol ? bad.as<int>() : nullptr);
      qr_form_u(dd.as<MatDesc>(), hc, snmax, s, true, nb);
      HIP_CHECK(hipEventRecord(e1, s));
      HIP_CHECK(hipEventSynchronize(e1));
      HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
    }
    report += " " + std::to_string(nb) + ": " + std::to_string(ms) + " ms";
    if (nb == 16 || ms < best_ms) { best = nb; best_ms = ms; }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  progress("QR panel width for %s: %d (%s)", key.c_str(), best, report.c_str());
  tune_store(key, best);
  return best;
}

// One 32-column panel at a time (the panel width of the pivoted QR's T
// factors), for callers that act between panels.
struct QRPanels32::Impl {
  BlockedQR<32> q;
  Impl(const MatDesc *d, const std::vector<MatDesc> &h) : q(d, h) {}
};
QRPanels32::QRPanels32(const MatDesc *descs, const std::vector<MatDesc> &h) : impl(new Impl(descs, h)) {}
QRPanels32::~QRPanels32() { delete impl; }
void QRPanels32::panel(int K0, hipStream_t s) { impl->q.panel(K0, s); }

void qr_factor(const MatDesc *descs, const std::vector<MatDesc> &h, hipStream_t s, int nb, int *bad) {
  switch (nb) {
    case 16: qr_factor_t<16>(descs, h, s, bad); break;
    case 32: qr_factor_t<32>(descs, h, s, bad); break;
    case 64: qr_factor_t<64>(descs, h, s, bad); break;
    default: MFS_THROW(MFS_EINVAL, "QR panel width must be 16, 32 or 64");
  }
}

// Form U = Q [U_R; 0] in place in d.u (leading dimension d.ldu, or d.lda if
// zero); rows >= n of d.u must be zero.  T of every panel (of width nb, the
// width the QR ran with) must be present.  from_identity: d.u holds the
// first rank columns of the identity, so the panel at k0 updates its
// columns k0 and later only.
//
// Forming U is all trailing-update work (no panel to factor), so it always
// runs with 64-column block reflectors, whatever width the QR ran with:
// for a QR of panels of 16 or 32 columns, T of every 64 consecutive
// reflectors is formed first from their Householder vectors and tau
// (V^H V and the forward recurrence, as bqr_t_kernel does after a panel)
// into a buffer of its own, and U is formed with those.
void qr_form_u(const MatDesc *descs, const std::vector<MatDesc> &h, int maxrank, hipStream_t s,
               bool from_identity, int nb) {
  MFS_REQUIRE(nb == 16 || nb == 32 || nb == 64, "QR panel width must be 16, 32 or 64");
  int nmax = 0, mmax = 0;
  for (const auto &d : h) {
    nmax = std::max(nmax, d.n);
    mmax = std::max(mmax, d.m);
  }
  const int nmat = (int)h.size();
  if (maxrank <= 0 || nmax == 0 || nmat == 0) return;
  if (nb == 64 || nmax <= nb) {
    switch (nb) {
      case 16: qr_form_u_t<16>(descs, h, maxrank, s, from_identity); break;
      case 32: qr_form_u_t<32>(descs, h, maxrank, s, from_identity); break;
      default: qr_form_u_t<64>(descs, h, maxrank, s, from_identity); break;
    }
    return;
  }
  std::vector<MatDesc> h2(h);
  std::vector<size_t> off(nmat);
  size_t tot = 0;
  for (int i = 0; i < nmat; ++i) {
    off[i] = tot;
    tot += (size_t)cdiv(std::max(h[i].n, 1), 64) * 64 * 64;
  }
  DevBuf t64(tot * sizeof(double2)), d2(nmat * sizeof(MatDesc));
  for (int i = 0; i < nmat; ++i) h2[i].T = t64.as<double2>() + off[i];
  HIP_CHECK(hipMemcpyAsync(d2.p, h2.data(), nmat * sizeof(MatDesc), hipMemcpyHostToDevice, s));
  {
    ApplyWork w;
    w.size(nmat, mmax, 0, 64);
    for (int k0 = 0; k0 < nmax; k0 += 64)   // V^H V of the group only (no trailing columns), then T
      apply_panel<64>(d2.as<MatDesc>(), nmat, mmax, 0, k0, 0, 1, 1, w, true, s, k0 + 64);
  }
  qr_form_u_t<64>(d2.as<MatDesc>(), h2, maxrank, s, from_identity);
}

}  // namespace mfs
