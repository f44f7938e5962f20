// Auxiliary spherical-harmonic basis H_lm = j_l(kr) Y_lm (eq. (urep)) and the
// Rayleigh-Bloch plane waves (eqs. (T)-(nD)): the per-incidence fill of
// Q = [S, -W] (Sec. 4.1), the Neumann data of the harmonics on the surface
// rings (the B~ block) and the harmonic part of the field at test points.
//
// Y_lm are orthonormal with the Condon-Shortley phase, Y_l^{-m} =
// (-1)^m conj(Y_l^m), origin at the obstacle centre.  Normalised associated
// Legendre functions by the standard stable recurrences
//   P_0^0 = 1/sqrt(4 pi),  P_m^m = -sqrt((2m+1)/(2m)) sin(th) P_{m-1}^{m-1},
//   P_{m+1}^m = sqrt(2m+3) cos(th) P_m^m,
//   P_l^m = a_lm (cos(th) P_{l-1}^m - b_lm P_{l-2}^m),
//   a_lm = sqrt((4l^2-1)/(l^2-m^2)), b_lm = sqrt(((l-1)^2-m^2)/(4(l-1)^2-1)),
// their theta derivative
//   dP_l^m/dth = (l cos(th) P_l^m - sqrt((2l+1)/(2l-1)) sqrt(l^2-m^2) P_{l-1}^m) / sin(th),
// and spherical Bessel functions by Miller's backward recurrence normalised
// with j_0 = sin x / x or j_1 = sin x / x^2 - cos x / x.  Cartesian gradients
// follow from grad H = dH/dr r^ + (1/r) dH/dth th^ + (1/(r sin th)) dH/dph ph^,
// so targets must lie off the z axis (wall nodes with M1 even, surface
// rings with rho > 0).
#include "internal.hpp"

namespace mfs {
namespace {

constexpr int MAXP = 96;

// j_l(x) and its derivative, l = 0..p, into j[l * ld], jp[l * ld]
__device__ void sph_bessel(int p, double x, double *j, double *jp, size_t ld) {
  const int L = p + 32 + (int)x;
  double fnext = 0.0, f = 1e-200;
  for (int l = L; l >= 1; --l) {
    const double fprev = (2.0 * l + 1.0) / x * f - fnext;   // f_{l-1}
    fnext = f;
    f = fprev;
    if (l - 1 <= p) j[(l - 1) * ld] = f;
    if (l <= p) j[l * ld] = fnext;
    if (fabs(f) > 1e250) {
      f *= 1e-250;
      fnext *= 1e-250;
      for (int i = l - 1; i <= p; ++i)
        if (i >= 0) j[i * ld] *= 1e-250;
    }
  }
  double s, c;
  sincos(x, &s, &c);
  const double j0 = s / x;
  const double j1 = s / (x * x) - c / x;
  double scale;
  if (fabs(j0) >= fabs(j1)) scale = j0 / j[0];
  else scale = j1 / j[ld];
  for (int l = 0; l <= p; ++l) j[l * ld] *= scale;
  jp[0] = -j[ld];
  for (int l = 1; l <= p; ++l) jp[l * ld] = j[(l - 1) * ld] - (l + 1.0) / x * j[l * ld];
}

// Spherical coordinates of a point and the frame vectors.
struct Sph {
  double r, ct, st, cp, sp;
};
__device__ inline Sph sph_of(double x, double y, double z) {
  Sph o;
  const double rho = sqrt(x * x + y * y);
  o.r = sqrt(rho * rho + z * z);
  o.ct = z / o.r;
  o.st = rho / o.r;
  o.cp = rho > 0.0 ? x / rho : 1.0;
  o.sp = rho > 0.0 ? y / rho : 0.0;
  return o;
}

// Visit l = m..p of one m >= 0: calls f(l, P_l^m, dP_l^m/dth).
template <class F>
__device__ inline void legendre_visit(int p, int m, double ct, double st, F f) {
  double pmm = 0.28209479177387814;   // 1/sqrt(4 pi)
  for (int i = 1; i <= m; ++i) pmm = -sqrt((2.0 * i + 1.0) / (2.0 * i)) * st * pmm;
  double p2 = 0.0, p1 = pmm;   // P_{l-2}, P_{l-1}
  f(m, pmm, (m * ct * pmm) / st);
  for (int l = m + 1; l <= p; ++l) {
    double pl;
    if (l == m + 1) pl = sqrt(2.0 * m + 3.0) * ct * pmm;
    else {
      const double a = sqrt((4.0 * l * l - 1.0) / ((double)l * l - (double)m * m));
      const double b = sqrt(((l - 1.0) * (l - 1.0) - (double)m * m) / (4.0 * (l - 1.0) * (l - 1.0) - 1.0));
      pl = a * (ct * p1 - b * p2);
    }
    const double dth = (l * ct * pl - sqrt((2.0 * l + 1.0) / (2.0 * l - 1.0)) *
                                          sqrt((double)l * l - (double)m * m) * p1) / st;
    f(l, pl, dth);
    p2 = p1;
    p1 = pl;
  }
}

__device__ inline int lm_col(int l, int m) { return l * l + l + m; }

// j_l(k r), j_l'(k r) of n points (SoA x, y, z; y null: 0) into j, jp [p+1][n]
__global__ __launch_bounds__(64) void bessel_table_kernel(int n, int p, double k, const double *x, const double *y,
                                                          const double *z, double *j, double *jp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  sph_bessel(p, k * sph_of(x[i], y ? y[i] : 0.0, z[i]).r, j + i, jp + i, n);
}

// S block of both halves of Q (QHalf in internal.hpp) for every wave: one
// thread per (node, m).  Bound by its stores (16 B x 4 (p + 1 - m) per wave):
// what a node contributes does not depend on the wave except for the Bloch
// phase, so a thread evaluates its harmonics once and writes them for all
// waves.  The nodes of a wall pair share radius, polar angle and, mirrored,
// azimuth: H_lm on L is (-1)^m conj(H_lm on R), on B conj(H_lm on F), and
// the normal derivatives change sign as well, so each pair is one evaluation.
// 8 waves of the k = 10 lattice (16 halves of 2304 x 650, 383 MB): 211 us, 28 us
// the table of Bessel functions before it; 1.88 ms with one thread per node
// and wave looping over all (l, m), both walls evaluated.
__global__ __launch_bounds__(64) void qfill_s_kernel(int W, int p, int M1, double k, const double *__restrict__ nodes,
                                                     const double *__restrict__ jt, const double *__restrict__ jpt,
                                                     const QFillArgs *__restrict__ args) {
  const int M1sq = M1 * M1, H = M1sq / 2, nn = 2 * M1sq;
  const int i = blockIdx.x * blockDim.x + threadIdx.x, m = blockIdx.y;
  if (i >= nn) return;
  const int unit = i < H ? 0 : (i < 2 * H ? 1 : 2);   // R/L, F/B, T/D
  const int rowv = unit == 0 ? i : (unit == 1 ? i + H : i + 2 * H);
  const int rowd = rowv + (unit == 2 ? M1sq : H);
  const Sph s = sph_of(nodes[i], nodes[nn + i], nodes[2 * nn + i]);
  double sm, cm;
  sincos(m * atan2(s.sp, s.cp), &sm, &cm);
  const double sg = (m & 1) ? -1.0 : 1.0;
  const double rt2 = 1.4142135623730951;
  // components of r^, th^, ph^ along the wall normal
  const double nr = unit == 0 ? s.st * s.cp : (unit == 1 ? s.st * s.sp : s.ct);
  const double nt = unit == 0 ? s.ct * s.cp : (unit == 1 ? s.ct * s.sp : -s.st);
  const double np = unit == 0 ? -s.sp : (unit == 1 ? s.cp : 0.0);
  const double msg = unit == 0 ? sg : 1.0;   // the mirrored wall: msg conj(.)
  legendre_visit(p, m, s.ct, s.st, [&](int l, double P, double dP) {
    const double jl = jt[(size_t)l * nn + i], jlp = jpt[(size_t)l * nn + i];
    // value e^{im phi} hv, derivative e^{im phi} (ga + i gb)
    const double hv = rt2 * jl * P;
    const double ga = rt2 * (k * jlp * P * nr + jl * dP / s.r * nt), gb = rt2 * m * jl * P / (s.r * s.st) * np;
    const double2 h = cz(hv * cm, hv * sm), g = cz(ga * cm - gb * sm, ga * sm + gb * cm);
    const int par = (l + m) & 1;
    const int base = par ? l * (l - 1) / 2 : l * (l + 1) / 2;
    const int cp = base + (l + m - par) / 2, cn = base + (l - m - par) / 2;
    for (int w = 0; w < W; ++w) {
      const QFillArgs a = args[w];
      double2 *Q = a.Q[par];
      double2 v = h, d = g, vn = cscale(cconj(h), sg), dn = cscale(cconj(g), sg);   // m and -m
      if (unit < 2) {
        const double2 ph = cscale(unit == 0 ? a.alpha : a.beta, msg);
        const double2 mv = cmul(ph, cconj(v)), md = cmul(ph, cconj(d));
        const double2 mvn = cmul(ph, cconj(vn)), mdn = cmul(ph, cconj(dn));
        v = csub(v, mv);
        d = cadd(d, md);
        vn = csub(vn, mvn);
        dn = cadd(dn, mdn);
      }
      Q[(size_t)cp * a.ldq + rowv] = v;
      Q[(size_t)cp * a.ldq + rowd] = d;
      if (m > 0) {
        Q[(size_t)cn * a.ldq + rowv] = vn;
        Q[(size_t)cn * a.ldq + rowd] = dn;
      }
    }
  });
}

// -W block of both halves: on T the plane waves (value -e, derivative
// -i kappa_z e), the same in the even and the odd half; zero on the side walls.
__global__ void qfill_w_kernel(int p, int M1, const double *__restrict__ nodes, const QFillArgs *__restrict__ args) {
  const QFillArgs a = args[blockIdx.y];   // one incidence per grid row
  const int M1sq = M1 * M1, H = M1sq / 2, nn = 2 * M1sq, rows = 4 * M1sq;
  const long total = (long)rows * a.nrb;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long)gridDim.x * blockDim.x) {
    const int o = (int)(idx / rows);
    const int row = (int)(idx % rows);
    double2 v = cz(0.0, 0.0);
    if (row >= 4 * H) {
      const int t = (row - 4 * H) % M1sq;
      double s, c;
      sincos(a.kx[o] * nodes[2 * H + t] + a.ky[o] * nodes[nn + 2 * H + t], &s, &c);
      v = cz(-c, -s);
      if (row - 4 * H >= M1sq) v = cmul(cz(-a.kz[o].y, a.kz[o].x), v);
    }
    a.Q[0][(size_t)((p + 1) * (p + 2) / 2 + o) * a.ldq + row] = v;
    a.Q[1][(size_t)(p * (p + 1) / 2 + o) * a.ldq + row] = v;
  }
}

// The wall sums (target groups of walls_plan, pad targets each) as right-hand
// sides of the two halves: out[2 w + par][row], rows_h rows, those past
// 4 M1^2 zero.
__global__ void split_walls_kernel(int nw, int M1, const double2 *__restrict__ in, double2 *__restrict__ out,
                                   int rows_h) {
  const int M1sq = M1 * M1, H = M1sq / 2, pad = (M1sq + 63) / 64 * 64;
  const long n = (long)nw * rows_h;
  const double rh = 0.70710678118654752;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int w = (int)(i / rows_h), row = (int)(i % rows_h);
    const double2 *src = in + (size_t)w * 12 * pad;
    double2 x = cz(0.0, 0.0), y = x;   // the node and its image under z -> -z
    double sg = 1.0;                   // the even half adds sg times the image
    if (row < 4 * H) {
      const int blk = row / H, e = row % H;
      const int t = e / (M1 / 2) * M1 + M1 / 2 + e % (M1 / 2);
      const int u = t / M1 * M1 + (M1 - 1 - t % M1);
      x = cadd(src[(2 * blk) * pad + t], src[(2 * blk + 1) * pad + t]);
      y = cadd(src[(2 * blk) * pad + u], src[(2 * blk + 1) * pad + u]);
    } else if (row < 4 * M1sq) {
      const int t = row - 4 * H, der = t >= M1sq ? 1 : 0;
      x = src[(8 + der) * pad + t - der * M1sq];
      y = src[(10 + der) * pad + t - der * M1sq];
      sg = der ? -1.0 : 1.0;
    }
    out[(size_t)(2 * w) * rows_h + row] = cz(rh * (x.x + sg * y.x), rh * (x.y + sg * y.y));
    out[(size_t)(2 * w + 1) * rows_h + row] = cz(rh * (x.x - sg * y.x), rh * (x.y - sg * y.y));
  }
}

// xi[w] in the column order of Q (harmonics l^2 + l + m, a, b) from the two
// halves' coefficients xh[2 w + par] (ldh apart)
__global__ void merge_xi_kernel(int nw, int p, const int *__restrict__ nrb, const double2 *__restrict__ xh, int ldh,
                                double2 *__restrict__ xi, int ldx) {
  const int w = blockIdx.y, NH = (p + 1) * (p + 1), nr = nrb[w];
  const double2 *e = xh + (size_t)(2 * w) * ldh, *o = e + ldh;
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < NH + 2 * nr; c += gridDim.x * blockDim.x) {
    double2 v;
    if (c < NH) {
      int l = (int)sqrt((double)c);
      if (l * l > c) --l;
      if ((l + 1) * (l + 1) <= c) ++l;
      const int lm = c - l * l;   // l + m
      v = (lm & 1) ? o[l * (l - 1) / 2 + (lm - 1) / 2] : e[l * (l + 1) / 2 + lm / 2];
    } else {
      const int q = (c - NH) % nr;
      const double2 ev = e[(p + 1) * (p + 2) / 2 + q], ov = o[p * (p + 1) / 2 + q];
      v = cscale(c - NH < nr ? cadd(ev, ov) : csub(ev, ov), 0.70710678118654752);
    }
    xi[(size_t)w * ldx + c] = v;
  }
}

__global__ void zero_kernel(double2 *p, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    p[i] = cz(0.0, 0.0);
}

// dH_lm/dn (value = 0) or H_lm at (rho_i, 0, z_i) with normal (nrho_i, 0,
// nz_i): out[lm][i], or, given, out_re[l (l + 1) / 2 + m][i] for m >= 0;
// one thread per (point, m); j, jp [p+1][M]
__global__ __launch_bounds__(64) void bfill_kernel(int M, int p, double k, const double *rho,
                                                   const double *z, const double *nrho,
                                                   const double *nz, const double *__restrict__ j,
                                                   const double *__restrict__ jp, double2 *out, double *out_re, int value) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x, m = blockIdx.y;
  if (i >= M) return;
  const Sph s = sph_of(rho[i], 0.0, z[i]);
  const double nr = value ? 0.0 : nrho[i], nzz = value ? 0.0 : nz[i];
  legendre_visit(p, m, s.ct, s.st, [&](int l, double P, double dP) {
    const double jl = j[(size_t)l * M + i];
    const double dr = k * jp[(size_t)l * M + i] * P, dth = jl * dP / s.r;
    // d/drho = st d/dr + ct/r d/dth ; d/dz = ct d/dr - st/r d/dth  (phi = 0)
    const double v = value ? jl * P : nr * (s.st * dr + s.ct * dth) + nzz * (s.ct * dr - s.st * dth);
    if (out_re) {
      out_re[((size_t)l * (l + 1) / 2 + m) * M + i] = v;
      return;
    }
    out[(size_t)lm_col(l, m) * M + i] = cz(v, 0.0);
    if (m > 0) out[(size_t)lm_col(l, -m) * M + i] = cz((m & 1) ? -v : v, 0.0);
  });
}

// out[r][b][i] -= sum over (l, mm) with mm = b (mod P) of B[lm][i] d[r][lm];
// out[r][b][i] at (r P + b) ldo + i
__global__ void bapply_kernel(int nrhs, int P, int M, int p, const double2 *__restrict__ B,
                              const double2 *__restrict__ d, int ldd, double2 *__restrict__ out, int ldo) {
  const long total = (long)nrhs * P * M;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long)gridDim.x * blockDim.x) {
    const int i = (int)(idx % M);
    const int b = (int)((idx / M) % P);
    const int r = (int)(idx / ((long)M * P));
    double2 acc = cz(0.0, 0.0);
    // modes mm congruent to b with |mm| <= p
    int mm0 = b;
    while (mm0 - P >= -p) mm0 -= P;   // smallest candidate >= -p
    for (int mm = mm0; mm <= p; mm += P) {
      const int am = mm < 0 ? -mm : mm;
      for (int l = am; l <= p; ++l) {
        const int col = lm_col(l, mm);
        cfma(acc, B[(size_t)col * M + i], d[(size_t)r * ldd + col]);
      }
    }
    const size_t o = ((size_t)r * P + b) * ldo + i;
    out[o] = csub(out[o], acc);
  }
}

// u[r][t] += sum_lm H_lm(x_t) d[r][lm]: one workgroup per target, one thread
// per m (a thread per target left all but one of the chip's wavefronts idle:
// 1.68 ms for 44 targets and 8 waves, 0.10 ms now for 32)
constexpr int HF = 128, HFR = 16;   // MAXP < HF
__global__ __launch_bounds__(HF) void harm_field_kernel(int nrhs, int nt, const double *xyz, int p,
                                                        double k, const double2 *d, int ldd,
                                                        double2 *out) {
  const int t = blockIdx.x, m = threadIdx.x;
  __shared__ double j[MAXP + 1], jp[MAXP + 1];
  __shared__ double2 red[HF / 64][HFR];
  const Sph s = sph_of(xyz[3 * t], xyz[3 * t + 1], xyz[3 * t + 2]);
  if (m == 0) sph_bessel(p, k * s.r, j, jp, 1);
  __syncthreads();
  double sm, cm;
  sincos(m * atan2(s.sp, s.cp), &sm, &cm);
  const double sg = (m & 1) ? -1.0 : 1.0;
  for (int r0 = 0; r0 < nrhs; r0 += HFR) {
    const int nr = min(HFR, nrhs - r0);
    double2 acc[HFR];
#pragma unroll
    for (int r = 0; r < HFR; ++r) acc[r] = cz(0.0, 0.0);
    if (m <= p)
      legendre_visit(p, m, s.ct, s.st, [&](int l, double P, double) {
        const double2 hv = cz(j[l] * P * cm, j[l] * P * sm), hn = cscale(cconj(hv), sg);
#pragma unroll
        for (int r = 0; r < HFR; ++r)
          if (r < nr) {
            const double2 *dr = d + (size_t)(r0 + r) * ldd + lm_col(l, 0);
            cfma(acc[r], hv, dr[m]);
            if (m > 0) cfma(acc[r], hn, dr[-m]);
          }
      });
#pragma unroll
    for (int r = 0; r < HFR; ++r) {
      const double2 v = wave_sum(acc[r]);
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][r] = v;
    }
    __syncthreads();
    if (m < nr) {
      double2 *o = out + (size_t)(r0 + m) * nt + t;
      *o = cadd(*o, cadd(red[0][m], red[1][m]));
    }
    __syncthreads();
  }
}

}  // namespace

// Nodes of the half system: R then F on the half z > 0 (b >= M1/2 of node
// (a, b)), then T; SoA x, y, z [2 M1^2] each, from the walls' SoA.
void half_nodes(int M1, const std::vector<double> &wall, std::vector<double> &out) {
  const int M1sq = M1 * M1, H = M1sq / 2, nn = 2 * M1sq;
  out.assign((size_t)3 * nn, 0.0);
  for (int c = 0; c < 3; ++c) {
    for (int e = 0; e < H; ++e) {
      const int t = e / (M1 / 2) * M1 + M1 / 2 + e % (M1 / 2);
      out[(size_t)c * nn + e] = wall[(size_t)c * M1sq + t];
      out[(size_t)c * nn + H + e] = wall[(size_t)(6 + c) * M1sq + t];
    }
    for (int t = 0; t < M1sq; ++t) out[(size_t)c * nn + 2 * H + t] = wall[(size_t)(12 + c) * M1sq + t];
  }
}

static void bessel_table(int n, int p, double k, const double *x, const double *y, const double *z, DevBuf &jt,
                         hipStream_t s) {
  jt.alloc((size_t)2 * (p + 1) * n * sizeof(double));
  double *j = jt.as<double>();
  hipLaunchKernelGGL(bessel_table_kernel, dim3(cdiv(n, 64)), dim3(64), 0, s, n, p, k, x, y, z, j,
                     j + (size_t)(p + 1) * n);
}

void launch_qfill(const std::vector<QFillArgs> &h, int p, int M1, int rows_h, double k, const double *nodes,
                  hipStream_t s) {
  const int W = (int)h.size();
  if (W == 0) return;
  MFS_REQUIRE(p <= MAXP, "harmonic degree p exceeds 96");
  const int nn = 2 * M1 * M1, rows = 4 * M1 * M1;
  int nrbmax = 0;
  for (const auto &a : h) {
    nrbmax = std::max(nrbmax, a.nrb);
    if (rows_h == rows) continue;
    for (int par = 0; par < 2; ++par) {   // more columns than rows: zero rows below (every other row is written)
      const long n = (long)a.ldq * ((par ? p * (p + 1) / 2 : (p + 1) * (p + 2) / 2) + a.nrb);
      hipLaunchKernelGGL(zero_kernel, dim3((unsigned)std::min<long>(4096, (n + 255) / 256)), dim3(256), 0, s,
                         a.Q[par], n);
    }
  }
  DevBuf args(h.size() * sizeof(QFillArgs)), jt;
  HIP_CHECK(hipMemcpyAsync(args.p, h.data(), h.size() * sizeof(QFillArgs), hipMemcpyHostToDevice, s));
  bessel_table(nn, p, k, nodes, nodes + nn, nodes + 2 * nn, jt, s);
  hipLaunchKernelGGL(qfill_s_kernel, dim3(cdiv(nn, 64), p + 1), dim3(64), 0, s, W, p, M1, k, nodes, jt.as<double>(),
                     jt.as<double>() + (size_t)(p + 1) * nn, args.as<QFillArgs>());
  const long nw = (long)rows * nrbmax;
  if (nw > 0)
    hipLaunchKernelGGL(qfill_w_kernel, dim3((unsigned)std::min<long>(4096, (nw + 255) / 256), W), dim3(256), 0, s, p,
                       M1, nodes, args.as<QFillArgs>());
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipStreamSynchronize(s));   // the argument array is released on return
}

void launch_split_walls(int nw, int M1, const double2 *in, double2 *out, int rows_h, hipStream_t s) {
  const long n = (long)nw * rows_h;
  hipLaunchKernelGGL(split_walls_kernel, dim3((unsigned)std::min<long>(1024, (n + 255) / 256)), dim3(256), 0, s, nw,
                     M1, in, out, rows_h);
  HIP_CHECK(hipGetLastError());
}

void launch_merge_xi(int nw, int p, int nqmax, const int *nrb, const double2 *xh, int ldh, double2 *xi, int ldx,
                     hipStream_t s) {
  hipLaunchKernelGGL(merge_xi_kernel, dim3(cdiv(nqmax, 256), nw), dim3(256), 0, s, nw, p, nrb, xh, ldh, xi, ldx);
  HIP_CHECK(hipGetLastError());
}

static void bfill(int M, int p, double k, const double *rho, const double *z, const double *nrho, const double *nz,
                  double2 *out, double *out_re, hipStream_t s, int value) {
  DevBuf jt;
  bessel_table(M, p, k, rho, nullptr, z, jt, s);
  hipLaunchKernelGGL(bfill_kernel, dim3(cdiv(M, 64), p + 1), dim3(64), 0, s, M, p, k, rho, z, nrho, nz,
                     jt.as<double>(), jt.as<double>() + (size_t)(p + 1) * M, out, out_re, value);
  HIP_CHECK(hipGetLastError());
}
void launch_bfill(int M, int p, double k, const double *rho, const double *z, const double *nrho,
                  const double *nz, double2 *out, hipStream_t s, int value) {
  bfill(M, p, k, rho, z, nrho, nz, out, nullptr, s, value);
}
void launch_bfill_real(int M, int p, double k, const double *rho, const double *z, const double *nrho,
                       const double *nz, double *out, hipStream_t s, int value) {
  bfill(M, p, k, rho, z, nrho, nz, nullptr, out, s, value);
}

void launch_bapply(int nrhs, int P, int M, int p, const double2 *B, const double2 *d, int ldd,
                   double2 *out, hipStream_t s, int ldo) {
  const long n = (long)nrhs * P * M;
  if (ldo <= 0) ldo = M;
  hipLaunchKernelGGL(bapply_kernel, dim3((unsigned)std::min<long>(2048, (n + 255) / 256)), dim3(256), 0, s,
                     nrhs, P, M, p, B, d, ldd, out, ldo);
  HIP_CHECK(hipGetLastError());
}

void launch_harm_field(int nrhs, int nt, const double *xyz, int p, double k, const double2 *d,
                       int ldd, double2 *out, hipStream_t s) {
  MFS_REQUIRE(p <= MAXP, "harmonic degree p exceeds 96");
  hipLaunchKernelGGL(harm_field_kernel, dim3(nt), dim3(HF), 0, s, nrhs, nt, xyz, p, k, d, ldd, out);
  HIP_CHECK(hipGetLastError());
}

}  // namespace mfs
