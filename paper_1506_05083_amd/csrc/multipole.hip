// Near-field sums by outgoing and regular spherical-wave expansions: the
// surface sums of A_else (eq. (A)) and the wall rows of C (eq. (full)).
//
// Addition theorem: the sources of one copy lie in a ball of radius a_s, so
// their field outside it is sum_lm M_lm h_l(k|x|) Y_lm(x) with
//   M_lm = i k sum_j j_l(k r_j) Y_lm(y_j at azimuth 0) c[m mod P][j]
// straight from the mode coefficients c (the P-angle point strengths of a
// ring sum to c at the bin of m).  On the surface of the central copy the
// eight neighbours' field is regular, sum_lm L_lm j_l(k|x|) Y_lm(x), and
//   L = T M,  T_{lm,l'm'} = sum_j 4 pi (-1)^((l + l' + j)/2 + l')
//             Gaunt(l'm', lm, j m'-m) S_{j,m'-m},
//   S_jm = sum_e alpha^a beta^b h_j(k|e|) Y_jm(-e)
// (the eight images summed once per wave).  Both steps keep the parity of
// l + m (the images lie in the plane z = 0), so T is two dense blocks, and the
// wall rows in the half system of the periodizer (internal.hpp) likewise: per
// wave and parity one matrix G = [T; C] takes the moments to the regular
// coefficients and to the right-hand side of Q^+ in one product.  The azimuth
// transforms of the point sums disappear: moments read mode bins, and the
// local expansion is evaluated in mode bins like B~ xi, with which it is added.
//
// The degrees are those at which the tail of sum (2l+1) j_l(k r<) h_l(k r>)
// falls below 1e-15 of 1 / (k r>) for the nearest source and target allowed by
// the bounding spheres; bodies that nearly fill the cell need too many and
// keep the stored kernel values (Solver::setup_sums).
#include <algorithm>
#include <cmath>

#include "geometry.hpp"
#include "internal.hpp"

namespace mfs {
namespace {

// w_img = alpha^a beta^b, |alpha| = |beta| = 1
__device__ inline double2 phase(double2 al, double2 be, int a, int b) {
  double2 v = cz(1.0, 0.0);
  if (a) v = a > 0 ? al : cconj(al);
  if (b) v = cmul(v, b > 0 ? be : cconj(be));
  return v;
}

// S_jm of every wave: S[w][j (j + 1) / 2 + (m + j) / 2], m = -j, -j + 2, .., j
// (the others vanish in the plane); hd[3][J + 1] = h_j at ex, ey and the
// diagonal.
__global__ void lattice_sum_kernel(int J, double ex, double ey, const double2 *__restrict__ hd,
                                   const ExpWave *__restrict__ waves, double2 *__restrict__ S) {
  const int nS = (J + 1) * (J + 2) / 2;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nS) return;
  const ExpWave wv = waves[blockIdx.y];
  int j = (int)((sqrt(8.0 * i + 1.0) - 1.0) * 0.5);
  while (j * (j + 1) / 2 > i) --j;
  while ((j + 1) * (j + 2) / 2 <= i) ++j;
  const int m = 2 * (i - j * (j + 1) / 2) - j, am = m < 0 ? -m : m;
  // P_j^|m|(0): the l = m value, then every second degree
  double P = 0.28209479177387814;
  for (int q = 1; q <= am; ++q) P *= -sqrt((2.0 * q + 1.0) / (2.0 * q));
  for (int l = am + 2; l <= j; l += 2) {
    const double a = sqrt((4.0 * l * l - 1.0) / ((double)l * l - (double)am * am));
    const double b = sqrt(((l - 1.0) * (l - 1.0) - (double)am * am) / (4.0 * (l - 1.0) * (l - 1.0) - 1.0));
    P *= -a * b;
  }
  if (m < 0 && (am & 1)) P = -P;
  double2 acc = cz(0.0, 0.0);
  for (int a = -1; a <= 1; ++a)
    for (int b = -1; b <= 1; ++b) {
      if (a == 0 && b == 0) continue;
      double s, c;
      sincos(m * atan2(-b * ey, -a * ex), &s, &c);
      const double2 h = hd[(a == 0 ? 1 : (b == 0 ? 0 : 2)) * (J + 1) + j];
      cfma(acc, cmul(phase(wv.alpha, wv.beta, a, b), cz(c * P, s * P)), h);
    }
  S[(size_t)blockIdx.y * nS + i] = acc;
}

// T blocks of one (l, l') and parity for WG waves.  A thread takes entries
// (m, m') and runs the three-term recurrence of the 3j symbols (l' l j;
// m' -m m-m') in j (Schulten and Gordon 1975) upwards from its smallest and
// downwards from its largest j to a middle j where both directions are stable,
// multiplying into the waves' lattice sums as it goes; the two runs are
// matched on two neighbouring j and normalised by sum (2j+1) f^2 = 1, so
// nothing is stored.  Bound by the recurrence (a step is one root and its
// reciprocal, the other quotients from tables in LDS: 485 -> 375 us for one k = 10
// wave, with a division and two roots a step before); the lattice sums are read coalesced, neighbouring lanes
// holding neighbouring m' - m.  Consecutive lanes are consecutive rows m of a
// column, the order T is stored in.
constexpr int XPMAX = kExpMaxDegree, XJ = 2 * XPMAX + 2;
template <int WG>
__global__ __launch_bounds__(256) void translation_kernel(int W, int J, ExpShape x, const double2 *__restrict__ S,
                                                          const ExpWave *__restrict__ waves) {
  const int lp = blockIdx.x, l = blockIdx.y, par = blockIdx.z & 1, w0 = (blockIdx.z >> 1) * WG;
  const int nr = par ? l : l + 1, nc = par ? lp : lp + 1;
  if (nr == 0 || nc == 0) return;
  __shared__ double ta[XJ], g0[XJ], tf[XJ], tb[XJ];
  const int jlo = l > lp ? l - lp : lp - l, jhi = l + lp;
  for (int j = jlo + threadIdx.x; j <= jhi + 1; j += 256) {
    const double d = (double)(l - lp), q = (double)(jhi + 1);
    ta[j] = sqrt(fmax(0.0, ((double)j * j - d * d) * (q * q - (double)j * j)));
  }
  __syncthreads();
  // 1 / (j a(j+1)) of the step up from j, 1 / ((j+1) a(j)) of the step down
  for (int j = jlo + threadIdx.x; j <= jhi; j += 256) {
    tf[j] = 1.0 / ((j == 0 ? 1.0 : (double)j) * ta[j + 1]);
    tb[j] = 1.0 / ((j + 1.0) * ta[j]);
  }
  if (threadIdx.x == 0) {   // |(l' l j; 0 0 0)| for even l + l' + j, times sqrt(4 pi (2l+1)(2l'+1)(2j+1))
    double f = 1.0, n = 0.0;
    for (int j = jlo; j <= jhi; j += 2) {
      g0[j] = f;
      n += (2.0 * j + 1.0) * f * f;
      if (j + 2 <= jhi) f *= ta[j + 1] / ta[j + 2];
    }
    n = sqrt(4.0 * kPi * (2.0 * l + 1.0) * (2.0 * lp + 1.0) / n);
    for (int j = jlo; j <= jhi; j += 2) g0[j] *= n * sqrt(2.0 * j + 1.0);
  }
  __syncthreads();
  const int nS = (J + 1) * (J + 2) / 2;
  const int rbase = par ? l * (l - 1) / 2 : l * (l + 1) / 2, cbase = par ? lp * (lp - 1) / 2 : lp * (lp + 1) / 2;
  const double2 *Sw[WG];
#pragma unroll
  for (int w = 0; w < WG; ++w) Sw[w] = S + (size_t)min(w0 + w, W - 1) * nS;
  const double c2 = lp * (lp + 1.0), c3 = l * (l + 1.0);
  for (int e = threadIdx.x; e < nr * nc; e += 256) {
    const int m = 2 * (e % nr) + par - l, mp = 2 * (e / nr) + par - lp;
    const int m1 = m - mp;                       // third projection of the symbol
    const int a1 = m1 < 0 ? -m1 : m1;
    const int jmin = max(jlo, a1);
    const double dm = (double)(-m - mp), fm1 = (double)m1;
    const double q1 = fm1 * fm1;
    const double mid = q1 + (double)(lp * lp - mp * mp) + (double)(l * l - m * m);
    const int jm = min(max((int)sqrt(mid), jmin), jhi - 1);
    double2 af[WG], ab[WG];
#pragma unroll
    for (int w = 0; w < WG; ++w) af[w] = ab[w] = cz(0.0, 0.0);
    double lam = 0.0, nf = 0.0, nb = 0.0;
    const int par_j = jhi & 1;
    auto add = [&](double2(&acc)[WG], int j, double f) {
      const double g = g0[j] * f;
      const int i = j * (j + 1) / 2 + (j - m1) / 2;   // projection m' - m = -m1
#pragma unroll
      for (int w = 0; w < WG; ++w) {
        const double2 sv = Sw[w][i];
        acc[w].x = fma(g, sv.x, acc[w].x);
        acc[w].y = fma(g, sv.y, acc[w].y);
      }
    };
    if (jmin == jhi) {
      nf = 2.0 * jhi + 1.0;
      lam = 1.0;
      add(af, jhi, 1.0);
    } else {
      // c(j) = sqrt(j^2 - m1^2);
      // j a(j+1) c(j+1) f(j+1) + B(j) f(j) + (j+1) a(j) c(j) f(j-1) = 0
      double f = 1.0, fprev = 0.0, ac = ta[jmin] * sqrt((double)jmin * jmin - q1);
      for (int j = jmin; j <= jm; ++j) {
        const double dj = (double)j;
        nf += (2.0 * dj + 1.0) * f * f;
        if ((j & 1) == par_j) add(af, j, f);
        double ci;
        const double acn = ta[j + 1] * dist((dj + 1.0) * (dj + 1.0) - q1, ci);
        double fn;
        if (j == 0) fn = -dm * f * (tf[0] * ci);
        else {
          const double B = -(2.0 * dj + 1.0) * ((c2 - c3) * fm1 - dj * (dj + 1.0) * dm);
          fn = -(B * f + (dj + 1.0) * ac * fprev) * (tf[j] * ci);
        }
        fprev = f;
        f = fn;
        ac = acn;
      }
      const double f0 = fprev, f1 = f;   // f(jm), f(jm + 1)
      double g = 1.0, gnext = 0.0;
      ac = 0.0;                          // a(jhi + 1) = 0
      for (int j = jhi; j > jm; --j) {
        const double dj = (double)j;
        nb += (2.0 * dj + 1.0) * g * g;
        if ((j & 1) == par_j) add(ab, j, g);
        double ci;
        const double acj = ta[j] * dist(dj * dj - q1, ci);
        const double B = -(2.0 * dj + 1.0) * ((c2 - c3) * fm1 - dj * (dj + 1.0) * dm);
        const double gn = -(B * g + dj * ac * gnext) * (tb[j] * ci);
        gnext = g;
        g = gn;
        ac = acj;
      }
      lam = (f0 * g + f1 * gnext) / (g * g + gnext * gnext);   // g = g(jm), gnext = g(jm + 1)
    }
    const double sc = ((par != 0) != (lam < 0.0) ? -1.0 : 1.0) / sqrt(nf + lam * lam * nb);
    const size_t at = (size_t)(cbase + e / nr) * x.ldg + rbase + e % nr;
#pragma unroll
    for (int w = 0; w < WG; ++w)
      if (w0 + w < W)
        waves[w0 + w].G[par][at] = cz(sc * (af[w].x + lam * ab[w].x), sc * (af[w].y + lam * ab[w].y));
  }
}

// h_l(k r) and h_l'(k r), l = 0..p, of the half-system nodes seen from the
// image centres: slot s of a node of R is the image (-1, s - 1), of F
// (s - 1, -1), of T (s / 3 - 1, s % 3 - 1); hk[s][l][i] = h, then h'.
__device__ inline void node_image(const double *__restrict__ nodes, int nn, int H, int i, int s, double ex, double ey,
                                  double &X, double &Y, double &Z) {
  const int unit = i < H ? 0 : (i < 2 * H ? 1 : 2);
  const int a = unit == 0 ? -1 : (unit == 1 ? s - 1 : s / 3 - 1), b = unit == 0 ? s - 1 : (unit == 1 ? -1 : s % 3 - 1);
  X = nodes[i] - a * ex;
  Y = nodes[nn + i] - b * ey;
  Z = nodes[2 * nn + i];
}
__global__ __launch_bounds__(64) void hankel_table_kernel(int nn, int H, int p, double k, double ex, double ey,
                                                          const double *__restrict__ nodes, double2 *__restrict__ hk,
                                                          double2 *__restrict__ hp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x, s = blockIdx.y;
  if (i >= nn || (i < 2 * H && s >= 3)) return;
  double X, Y, Z;
  node_image(nodes, nn, H, i, s, ex, ey, X, Y, Z);
  const double x = k * sqrt(X * X + Y * Y + Z * Z);
  double2 *h = hk + (size_t)s * (p + 1) * nn + i, *d = hp + (size_t)s * (p + 1) * nn + i;
  // j_l downwards (Miller), y_l upwards
  const int L = p + 32 + (int)x;
  double fnext = 0.0, f = 1e-200;
  for (int l = L; l >= 1; --l) {
    const double fprev = (2.0 * l + 1.0) / x * f - fnext;
    fnext = f;
    f = fprev;
    if (l - 1 <= p) h[(size_t)(l - 1) * nn].x = f;
    if (l <= p) h[(size_t)l * nn].x = fnext;
    if (fabs(f) > 1e250) {
      f *= 1e-250;
      fnext *= 1e-250;
      for (int q = max(0, l - 1); q <= p; ++q) h[(size_t)q * nn].x *= 1e-250;
    }
  }
  double sn, cn;
  sincos(x, &sn, &cn);
  const double j0 = sn / x, j1 = sn / (x * x) - cn / x;
  const double scale = fabs(j0) >= fabs(j1) ? j0 / h[0].x : j1 / h[nn].x;
  double y0 = -cn / x, y1 = -cn / (x * x) - sn / x;
  double2 prev = cz(0.0, 0.0);
  for (int l = 0; l <= p; ++l) {
    const double2 v = cz(h[(size_t)l * nn].x * scale, y0);
    h[(size_t)l * nn] = v;
    // h_0' = -h_1: j1 and y1 in closed form
    d[(size_t)l * nn] = l == 0 ? cz(-j1, -y1) : cz(prev.x - (l + 1.0) / x * v.x, prev.y - (l + 1.0) / x * v.y);
    const double yn = (2.0 * l + 3.0) / x * y1 - y0;
    y0 = y1;
    y1 = yn;
    prev = v;
  }
}

// Wall rows of G for WG waves: one thread per (node, m >= 0), looping over l
// with the Legendre values of all the node's images carried along, and writing
// the columns m and -m.  SIDE: the pairs R - alpha L and F - beta B with the
// three images the 3x3 cancellation leaves; the partner wall's node sees the
// opposite image from the mirrored direction, so its radial and polar parts are
// the same.  Otherwise T with nine images.  45 us (side walls) and 145 us (T)
// for 8 waves at k = 10, 24 x 24 nodes a wall, degrees 23 and 36.
template <bool SIDE, int WG>
__global__ __launch_bounds__(64) void wall_rows_kernel(int W, double k, double ex, double ey, ExpShape x, int ptab,
                                                       const double *__restrict__ nodes,
                                                       const double2 *__restrict__ hk, const double2 *__restrict__ hp,
                                                       const ExpWave *__restrict__ waves) {
  constexpr int NI = SIDE ? 3 : 9;
  const int H = x.M1 * x.M1 / 2, nn = 4 * H;
  const int i = blockIdx.x * 64 + threadIdx.x + (SIDE ? 0 : 2 * H), m = blockIdx.y, w0 = blockIdx.z * WG;
  if (i >= (SIDE ? 2 * H : nn)) return;
  const int unit = i < H ? 0 : (i < 2 * H ? 1 : 2), p = x.pw[unit];
  if (m > p) return;
  const int rowv = x.row0 + (unit == 0 ? i : (unit == 1 ? i + H : i + 2 * H));
  const int rowd = rowv + (unit == 2 ? 2 * H : H);
  const double sg = (m & 1) ? -1.0 : 1.0, msg = unit == 0 ? sg : 1.0, rt2 = 1.4142135623730951;
  double ct[NI], st[NI], ir[NI], p1[NI], p2[NI], cr[NI], cth[NI], cph[NI];
  double2 E[NI];
  double pm = 0.28209479177387814;
  for (int q = 1; q <= m; ++q) pm *= -sqrt((2.0 * q + 1.0) / (2.0 * q));
#pragma unroll
  for (int s = 0; s < NI; ++s) {
    double X, Y, Z;
    node_image(nodes, nn, H, i, s, ex, ey, X, Y, Z);
    const double rho = sqrt(X * X + Y * Y), r = sqrt(rho * rho + Z * Z);
    ct[s] = Z / r;
    st[s] = rho / r;
    ir[s] = 1.0 / r;
    const double cp = rho > 0.0 ? X / rho : 1.0, sp = rho > 0.0 ? Y / rho : 0.0;
    double sn, cn;
    sincos(m * atan2(sp, cp), &sn, &cn);
    E[s] = cz(cn, sn);
    cr[s] = unit == 0 ? st[s] * cp : (unit == 1 ? st[s] * sp : ct[s]);
    cth[s] = (unit == 0 ? ct[s] * cp : (unit == 1 ? ct[s] * sp : -st[s])) / (r * st[s]);
    cph[s] = SIDE ? m * (unit == 0 ? -sp : cp) / (r * st[s]) : 0.0;
    double sm = rt2 * pm;
    for (int q = 0; q < m; ++q) sm *= st[s];
    p1[s] = sm;   // P_m^m times sqrt 2
    p2[s] = 0.0;
  }
  for (int l = m; l <= p; ++l) {
    double a = 0.0, b = 0.0;
    if (l == m + 1) a = sqrt(2.0 * m + 3.0);
    else if (l > m) {
      a = sqrt((4.0 * l * l - 1.0) / ((double)l * l - (double)m * m));
      b = sqrt(((l - 1.0) * (l - 1.0) - (double)m * m) / (4.0 * (l - 1.0) * (l - 1.0) - 1.0));
    }
    const double e1 = l > m ? sqrt((2.0 * l + 1.0) / (2.0 * l - 1.0)) * sqrt((double)l * l - (double)m * m) : 0.0;
    double2 v[WG], d[WG], vn[WG], dn[WG];
#pragma unroll
    for (int w = 0; w < WG; ++w) v[w] = d[w] = vn[w] = dn[w] = cz(0.0, 0.0);
#pragma unroll
    for (int s = 0; s < NI; ++s) {
      double P = p1[s], pd = 0.0;   // pd: P_{l-1}
      if (l > m) {
        pd = p1[s];
        P = a * (ct[s] * p1[s] - b * p2[s]);
        p2[s] = p1[s];
        p1[s] = P;
      }
      const double dP = l * ct[s] * P - e1 * pd;   // sin(theta) dP/dtheta
      const double2 h = hk[((size_t)s * (ptab + 1) + l) * nn + i], hd = hp[((size_t)s * (ptab + 1) + l) * nn + i];
      const double2 hv = cscale(h, P);
      const double2 A = cadd(cscale(hd, k * P * cr[s]), cscale(h, dP * cth[s])), B = cscale(h, P * cph[s]);
      const double2 Ep = E[s], En = cconj(E[s]);
      // angular part e^{im phi}, and its mirror image e^{-im phi}
      const double2 vp = cmul(Ep, hv), vm = cmul(En, hv);
      const double2 dp = cmul(Ep, cz(A.x - B.y, A.y + B.x)), dm = cmul(En, cz(A.x + B.y, A.y - B.x));
      const int ia = unit == 0 ? -1 : (unit == 1 ? s - 1 : s / 3 - 1);
      const int ib = unit == 0 ? s - 1 : (unit == 1 ? -1 : s % 3 - 1);
#pragma unroll
      for (int w = 0; w < WG; ++w) {
        const ExpWave &wv = waves[min(w0 + w, W - 1)];
        const double2 u = phase(wv.alpha, wv.beta, ia, ib);
        cfma(v[w], u, vp);
        cfma(d[w], u, dp);
        cfma(vn[w], u, vm);
        cfma(dn[w], u, dm);
        if (SIDE) {   // the partner wall's image, times -alpha or -beta
          const double2 ph = unit == 0 ? wv.alpha : wv.beta;
          double2 t = cmul(ph, unit == 0 ? phase(wv.alpha, wv.beta, 1, ib) : phase(wv.alpha, wv.beta, ia, 1));
          t = cscale(t, msg);
          cfma(v[w], cscale(t, -1.0), vm);
          cfma(d[w], t, dm);
          cfma(vn[w], cscale(t, -1.0), vp);
          cfma(dn[w], t, dp);
        }
      }
    }
    const int par = (l + m) & 1, base = par ? l * (l - 1) / 2 : l * (l + 1) / 2;
    const size_t cp = (size_t)(base + (l + m - par) / 2) * x.ldg, cn = (size_t)(base + (l - m - par) / 2) * x.ldg;
#pragma unroll
    for (int w = 0; w < WG; ++w) {
      if (w0 + w >= W) continue;
      double2 *G = waves[w0 + w].G[par];
      G[cp + rowv] = v[w];
      G[cp + rowd] = d[w];
      if (m > 0) {
        G[cn + rowv] = cscale(vn[w], sg);
        G[cn + rowd] = cscale(dn[w], sg);
      }
    }
  }
}

// Moments of every wave from its mode coefficients c[w][P][ldc]: one wave of
// lanes per (l, m >= 0), lanes over the sources, WG incident waves together.
// out[2 w + parity][ldx], (l, m) in the halves' column order.  13 us for 8
// waves, degree 43, 200 sources (the angle transform and the 8 x 12800 point
// strengths it replaces: 40 us).
template <int WG>
__global__ __launch_bounds__(256) void moments_kernel(int W, int P, int N, int pm, double k,
                                                      const double *__restrict__ tab, const double2 *__restrict__ c,
                                                      int ldc, double2 *__restrict__ out, int ldx) {
  const int id = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, w0 = blockIdx.y * WG;
  if (id >= (pm + 1) * (pm + 2) / 2) return;
  int l = (int)((sqrt(8.0 * id + 1.0) - 1.0) * 0.5);
  while (l * (l + 1) / 2 > id) --l;
  while ((l + 1) * (l + 2) / 2 <= id) ++l;
  const int m = id - l * (l + 1) / 2;
  const int bp = m % P, bn = (P - bp) % P;
  double2 ap[WG], an[WG];
#pragma unroll
  for (int w = 0; w < WG; ++w) ap[w] = an[w] = cz(0.0, 0.0);
  for (int j = lane; j < N; j += 64) {
    const double t = tab[(size_t)id * N + j];
#pragma unroll
    for (int w = 0; w < WG; ++w) {
      const double2 *cw = c + (size_t)min(w0 + w, W - 1) * P * ldc;
      const double2 x = cw[(size_t)bp * ldc + j], y = cw[(size_t)bn * ldc + j];
      ap[w].x = fma(t, x.x, ap[w].x);
      ap[w].y = fma(t, x.y, ap[w].y);
      an[w].x = fma(t, y.x, an[w].x);
      an[w].y = fma(t, y.y, an[w].y);
    }
  }
  const int par = (l + m) & 1, base = par ? l * (l - 1) / 2 : l * (l + 1) / 2;
  const double sg = (m & 1) ? -k : k;
#pragma unroll
  for (int w = 0; w < WG; ++w) {
    const double2 x = wave_sum(ap[w]), y = wave_sum(an[w]);
    if (lane == 0 && w0 + w < W) {
      double2 *o = out + (size_t)(2 * (w0 + w) + par) * ldx + base;
      o[(l + m - par) / 2] = cz(-k * x.y, k * x.x);
      if (m > 0) o[(l - m - par) / 2] = cz(-sg * y.y, sg * y.x);
    }
  }
}

// columns of G that row `row` of a half uses
__device__ __host__ inline int exp_row_cols(const ExpShape &x, int row, int par) {
  auto half = [&](int p) { return par ? p * (p + 1) / 2 : (p + 1) * (p + 2) / 2; };
  const int H = x.M1 * x.M1 / 2;
  if (row < x.row0) return row < half(x.pt) ? half(x.ps) : 0;
  const int r = row - x.row0;
  if (r >= 8 * H) return 0;
  return half(x.pw[r < 2 * H ? 0 : (r < 4 * H ? 1 : 2)]);
}

// out[mat] = G[mat] x[mat] for every wave and parity (mat = 2 w + parity;
// G null: zeros).  A matrix-vector product bound by reading G once from HBM:
// 64 rows a workgroup, the four wavefronts take alternate runs of eight columns
// (eight 1 KB loads in flight each), x through scalar loads; the columns are
// split over gridDim.y workgroups where the rows alone leave the chip idle.
// 139 us for the 576 MB of 8 waves at k = 10 (4.15 TB/s).
__global__ __launch_bounds__(256) void exp_gemv_kernel(ExpShape x, const ExpWave *__restrict__ waves,
                                                       const double2 *__restrict__ xv, int ldx,
                                                       double2 *__restrict__ out, int ldo, int chunk) {
  const int mat = blockIdx.z, par = mat & 1;
  const double2 *G = waves[mat >> 1].G[par];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = blockIdx.x * 64 + lane;
  const int lim = G ? exp_row_cols(x, row, par) : 0;
  const int c0 = blockIdx.y * chunk, c1 = c0 + chunk;
  const double2 *xm = xv + (size_t)mat * ldx;
  const double2 *g = G + row;
  double2 acc = cz(0.0, 0.0), acc2 = acc;
  for (int q = c0 + 8 * wv; q < c1; q += 32) {
    if (!__any(q < lim)) break;
    if (q + 8 <= c1 && __all(q + 8 <= lim)) {
      double2 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = g[(size_t)(q + u) * x.ldg];
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        cfma(acc, v[u], xm[q + u]);
        cfma(acc2, v[u + 1], xm[q + u + 1]);
      }
    } else {
      for (int u = 0; u < 8; ++u)
        if (q + u < c1 && q + u < lim) cfma(acc, g[(size_t)(q + u) * x.ldg], xm[q + u]);
    }
  }
  __shared__ double2 part[4][64];
  part[wv][lane] = cadd(acc, acc2);
  __syncthreads();
  if (wv == 0 && row < ldo)
    out[((size_t)blockIdx.y * gridDim.z + mat) * ldo + row] =
        cadd(cadd(part[0][lane], part[1][lane]), cadd(part[2][lane], part[3][lane]));
}

__global__ void exp_reduce_kernel(long n, int nsplit, const double2 *__restrict__ part, double2 *__restrict__ out) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    double2 t = part[i];
    for (int s = 1; s < nsplit; ++s) t = cadd(t, part[(size_t)s * n + i]);
    out[i] = t;
  }
}

// out[w][b][i] = x[w][b][i] + sum over (l, m), m = b (mod P), of
// B_lm(i) (L_lm - xi_lm): the regular part of the neighbours' field and the
// periodizer's harmonics on the surface rings, in mode bins.  Rows [0, M) of a
// bin read tab, rows [M, 2M) tab2 (transmission).  64 rows a workgroup, its
// four wavefronts take every fourth l, WG incident waves together.  26 us for 8
// waves at k = 10 (the sums' angle transform, the addition and B~ xi: 60 us).
template <int WG>
__global__ __launch_bounds__(256) void local_kernel(int W, int P, int M, int pt, int pq, const double *__restrict__ tab,
                                                    const double *__restrict__ tab2, const double2 *__restrict__ Lc,
                                                    int ldl, const double2 *__restrict__ xi, int ldxi,
                                                    const double2 *__restrict__ xin, double2 *__restrict__ out) {
  const int Mr = tab2 ? 2 * M : M;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = blockIdx.x * 64 + lane, b = blockIdx.y, w0 = blockIdx.z * WG;
  const int ii = min(i, Mr - 1);
  const double *t = (ii < M ? tab : tab2 - M) + ii;
  const int pb = max(pt, pq);
  double2 acc[WG];
#pragma unroll
  for (int w = 0; w < WG; ++w) acc[w] = cz(0.0, 0.0);
  int m0 = b;
  while (m0 - P >= -pb) m0 -= P;   // smallest m = b (mod P), >= -pb
  for (int m = m0; m <= pb; m += P) {
    const int am = m < 0 ? -m : m;
    const double sg = (m < 0 && (am & 1)) ? -1.0 : 1.0;
    for (int l = am + wv; l <= pb; l += 4) {
      const double bv = sg * t[(size_t)(l * (l + 1) / 2 + am) * M];
      const int par = (l + am) & 1, q = (par ? l * (l - 1) / 2 : l * (l + 1) / 2) + (l + m - par) / 2;
#pragma unroll
      for (int w = 0; w < WG; ++w) {
        const size_t mat = 2 * (size_t)min(w0 + w, W - 1) + par;
        double2 d = cz(0.0, 0.0);
        if (l <= pt) d = Lc[mat * ldl + q];
        if (l <= pq) d = csub(d, xi[mat * ldxi + q]);
        acc[w].x = fma(bv, d.x, acc[w].x);
        acc[w].y = fma(bv, d.y, acc[w].y);
      }
    }
  }
  __shared__ double2 part[4][WG][64];
#pragma unroll
  for (int w = 0; w < WG; ++w) part[wv][w][lane] = acc[w];
  __syncthreads();
  for (int w = wv; w < WG; w += 4)
    if (i < Mr && w0 + w < W) {
      const size_t o = ((size_t)(w0 + w) * P + b) * Mr + i;
      out[o] = cadd(xin[o], cadd(cadd(part[0][w][lane], part[1][w][lane]), cadd(part[2][w][lane], part[3][w][lane])));
    }
}

// h_l(x), l = 0..p, on the host (j by Miller's recurrence, y upwards)
void host_hankel(int p, double x, std::vector<double2> &h) {
  const int L = p + 40 + (int)x;
  std::vector<double> j(L + 2, 0.0);
  j[L] = 1e-200;
  for (int l = L; l >= 1; --l) {
    j[l - 1] = (2.0 * l + 1.0) / x * j[l] - j[l + 1];
    if (std::fabs(j[l - 1]) > 1e200)
      for (int q = l - 1; q <= L; ++q) j[q] *= 1e-200;
  }
  const double j0 = std::sin(x) / x, j1 = std::sin(x) / (x * x) - std::cos(x) / x;
  const double sc = std::fabs(j0) >= std::fabs(j1) ? j0 / j[0] : j1 / j[1];
  double y0 = -std::cos(x) / x, y1 = -std::cos(x) / (x * x) - std::sin(x) / x;
  h.resize(p + 1);
  for (int l = 0; l <= p; ++l) {
    h[l] = cz(j[l] * sc, y0);
    const double yn = (2.0 * l + 3.0) / x * y1 - y0;
    y0 = y1;
    y1 = yn;
  }
}

// Smallest p with sum_{l > p} (2l+1) |j_l(k a) h_l(k D)| k D <= 1e-15, or -1
// if none up to the library's bound (or the magnitudes leave double's range:
// the tail starts at degree 120, where h_l(k D) does below k D of about 0.23,
// and the point sums stay for such long waves).
int expansion_degree(double k, double a, double D) {
  if (!(a > 0.0) || !(D > 1.05 * a)) return -1;
  const int L = 120;
  std::vector<double2> hs, hl;
  host_hankel(L, k * a, hs);
  host_hankel(L, k * D, hl);
  double tail = 0.0;
  for (int l = L; l > 0; --l) {
    const double t = (2.0 * l + 1.0) * std::fabs(hs[l].x) * std::hypot(hl[l].x, hl[l].y) * k * D;
    if (!std::isfinite(t) || (l == L && t > 1e-16)) return -1;
    tail += t;
    if (tail > 1e-15) return l <= kExpMaxDegree ? l : -1;
  }
  return 1;
}

// (l, m >= 0) table of j_l Y_lm (value) or its normal derivative on rings at azimuth 0
void ring_table(int n, int p, double k, const double *rho, const double *z, const double *nrho, const double *nz,
                int value, DevBuf &out, hipStream_t s) {
  out.alloc((size_t)(p + 1) * (p + 2) / 2 * n * sizeof(double));
  launch_bfill_real(n, p, k, rho, z, nrho, nz, out.as<double>(), s, value);
}

}  // namespace

bool NearExpansion::plan(const BodyData &b, const mfs_lattice &lat) {
  double at = 0.0, as = 0.0;
  for (int i = 0; i < b.M; ++i) at = std::max(at, std::hypot(b.h_rho[i], b.h_z[i]));
  for (int j = 0; j < b.N; ++j) as = std::max(as, std::hypot(b.h_srho[j], b.h_sz[j]));
  const double d = std::min(lat.ex, lat.ey);
  x = ExpShape{};
  x.M1 = lat.M1;
  x.ps = expansion_degree(b.k, as, d - at);
  x.pt = expansion_degree(b.k, at, d - as);
  x.pw[0] = expansion_degree(b.k, as, 1.5 * lat.ex);
  x.pw[1] = expansion_degree(b.k, as, 1.5 * lat.ey);
  x.pw[2] = expansion_degree(b.k, as, lat.z0);
  pm = x.ps;
  for (int u = 0; u < 3; ++u) {
    if (x.pw[u] < 0) return false;
    pm = std::max(pm, x.pw[u]);
  }
  if (x.ps < 0 || x.pt < 0) return false;
  k = b.k;
  ex = lat.ex;
  ey = lat.ey;
  P = b.P;
  M = b.M;
  N = b.N;
  pq = lat.p;
  std::vector<double2> h;
  host_hankel(x.ps + x.pt, k * d, h);
  const double top = std::hypot(h.back().x, h.back().y);
  if (!(top < 1e290)) return false;
  x.row0 = round_up(half_cols(x.pt, 0), 16);
  rows = x.row0 + 4 * lat.M1 * lat.M1;
  x.ldg = round_up(rows, 64);
  ldx = half_cols(pm, 0);
  wave_elems = (size_t)x.ldg * (half_cols(pm, 0) + half_cols(pm, 1));
  bytes_read = 0.0;
  for (int par = 0; par < 2; ++par)
    for (int r = 0; r < rows; ++r) bytes_read += 16.0 * exp_row_cols(x, r, par);
  return true;
}

void NearExpansion::setup(const BodyData &b, const mfs_lattice &lat, hipStream_t s) {
  std::vector<double> wall, hn;
  wall_nodes(lat, wall);
  half_nodes(lat.M1, wall, hn);
  nodes.alloc(hn.size() * sizeof(double));
  HIP_CHECK(hipMemcpyAsync(nodes.p, hn.data(), hn.size() * sizeof(double), hipMemcpyHostToDevice, s));
  ring_table(N, pm, k, b.srho, b.sz, nullptr, nullptr, 1, src_tab, s);
  const int pb = std::max(x.pt, pq);
  if (b.trans()) {
    ring_table(M, pb, k, b.rho, b.z, b.nrho, b.nz, 1, tab, s);
    ring_table(M, pb, k, b.rho, b.z, b.nrho, b.nz, 0, tab2, s);
  } else {
    ring_table(M, pb, k, b.rho, b.z, b.nrho, b.nz, 0, tab, s);
  }
  const int J = x.ps + x.pt;
  std::vector<double2> hd, h;
  for (double d : {ex, ey, std::hypot(ex, ey)}) {
    host_hankel(J, k * d, h);
    hd.insert(hd.end(), h.begin(), h.end());
  }
  hdist.alloc(hd.size() * sizeof(double2));
  HIP_CHECK(hipMemcpyAsync(hdist.p, hd.data(), hd.size() * sizeof(double2), hipMemcpyHostToDevice, s));
  const int H = x.M1 * x.M1 / 2, nn = 4 * H, p = std::max(x.pw[0], std::max(x.pw[1], x.pw[2]));
  hank.alloc((size_t)2 * 9 * (p + 1) * nn * sizeof(double2));
  hipLaunchKernelGGL(hankel_table_kernel, dim3(cdiv(nn, 64), 9), dim3(64), 0, s, nn, H, p, k, ex, ey, nodes.as<double>(),
                     hank.as<double2>(), hank.as<double2>() + (size_t)9 * (p + 1) * nn);
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipStreamSynchronize(s));   // hd goes out of scope
}

void NearExpansion::build(const std::vector<ExpWave> &h, hipStream_t s) const {
  const int W = (int)h.size(), J = x.ps + x.pt, nS = (J + 1) * (J + 2) / 2;
  if (W == 0) return;
  DevBuf waves((size_t)W * sizeof(ExpWave)), S((size_t)W * nS * sizeof(double2));
  const ExpWave *wv = waves.as<ExpWave>();
  HIP_CHECK(hipMemcpyAsync(waves.p, h.data(), W * sizeof(ExpWave), hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(lattice_sum_kernel, dim3(cdiv(nS, 256), W), dim3(256), 0, s, J, ex, ey, hdist.as<double2>(), wv,
                     S.as<double2>());
  if (W <= 2)
    hipLaunchKernelGGL(translation_kernel<2>, dim3(x.ps + 1, x.pt + 1, 2), dim3(256), 0, s, W, J, x, S.as<double2>(),
                       wv);
  else
    hipLaunchKernelGGL(translation_kernel<8>, dim3(x.ps + 1, x.pt + 1, 2 * cdiv(W, 8)), dim3(256), 0, s, W, J, x,
                       S.as<double2>(), wv);
  const int H = x.M1 * x.M1 / 2, nn = 4 * H, p = std::max(x.pw[0], std::max(x.pw[1], x.pw[2]));
  const double2 *hk = hank.as<double2>(), *hp = hk + (size_t)9 * (p + 1) * nn;
  hipLaunchKernelGGL((wall_rows_kernel<true, 2>), dim3(cdiv(2 * H, 64), std::max(x.pw[0], x.pw[1]) + 1, cdiv(W, 2)),
                     dim3(64), 0, s, W, k, ex, ey, x, p, nodes.as<double>(), hk, hp, wv);
  hipLaunchKernelGGL((wall_rows_kernel<false, 2>), dim3(cdiv(2 * H, 64), x.pw[2] + 1, cdiv(W, 2)), dim3(64), 0, s, W,
                     k, ex, ey, x, p, nodes.as<double>(), hk, hp, wv);
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipStreamSynchronize(s));   // h and the work buffers go out of scope
}

void NearExpansion::moments(int W, const double2 *c, int ldc, double2 *out, hipStream_t s) const {
  const int nlm = (pm + 1) * (pm + 2) / 2;
  if (W <= 2)
    hipLaunchKernelGGL(moments_kernel<2>, dim3(cdiv(nlm, 4), cdiv(W, 2)), dim3(256), 0, s, W, P, N, pm, k,
                       src_tab.as<double>(), c, ldc, out, ldx);
  else
    hipLaunchKernelGGL(moments_kernel<4>, dim3(cdiv(nlm, 4), cdiv(W, 4)), dim3(256), 0, s, W, P, N, pm, k,
                       src_tab.as<double>(), c, ldc, out, ldx);
  HIP_CHECK(hipGetLastError());
}

int NearExpansion::splits(int W) const {
  // workgroups of 64 rows; at least about eight a compute unit
  return std::max(1, std::min(16, 2048 / std::max(1, 2 * W * cdiv(rows, 64))));
}

void NearExpansion::apply(int W, const ExpWave *waves, const double2 *xm, double2 *out, int ldo, double2 *part,
                          hipStream_t s) const {
  const int ns = splits(W), chunk = round_up(cdiv(ldx, ns), 32);
  hipLaunchKernelGGL(exp_gemv_kernel, dim3(cdiv(ldo, 64), ns, 2 * W), dim3(256), 0, s, x, waves, xm, ldx,
                     ns > 1 ? part : out, ldo, chunk);
  if (ns > 1) {
    const long n = (long)2 * W * ldo;
    hipLaunchKernelGGL(exp_reduce_kernel, dim3((unsigned)std::min<long>(1024, (n + 255) / 256)), dim3(256), 0, s, n,
                       ns, part, out);
  }
  HIP_CHECK(hipGetLastError());
}

void NearExpansion::local(int W, const double2 *Lc, int ldl, const double2 *xi, int ldxi, const double2 *xin,
                          double2 *out, hipStream_t s) const {
  const int Mr = tab2.p ? 2 * M : M;
  if (W <= 2)
    hipLaunchKernelGGL(local_kernel<2>, dim3(cdiv(Mr, 64), P, cdiv(W, 2)), dim3(256), 0, s, W, P, M, x.pt, pq,
                       tab.as<double>(), tab2.as<double>(), Lc, ldl, xi, ldxi, xin, out);
  else
    hipLaunchKernelGGL(local_kernel<4>, dim3(cdiv(Mr, 64), P, cdiv(W, 4)), dim3(256), 0, s, W, P, M, x.pt, pq,
                       tab.as<double>(), tab2.as<double>(), Lc, ldl, xi, ldxi, xin, out);
  HIP_CHECK(hipGetLastError());
}

}  // namespace mfs
