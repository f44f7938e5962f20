// Shared helpers of libmfs: complex double arithmetic on double2, error
// reporting across the C ABI, and small device utilities (wave64 reductions).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <string>

#include "../../include/mfs.h"

namespace mfs {

// ------------------------------------------------------------ errors
void set_error(const std::string &msg);
const std::string &get_error();

// Stage progress on stderr when the environment sets MFS_PROGRESS (long
// solves report what they are doing; printf-style, one line, flushed).
void progress(const char *fmt, ...);

struct Error {
  mfs_status st;
  std::string msg;
};

#define MFS_THROW(code, msg_expr)                                                 \
  do {                                                                            \
    throw ::mfs::Error{(code), std::string(msg_expr)};                            \
  } while (0)

#define HIP_CHECK(expr)                                                           \
  do {                                                                            \
    hipError_t e_ = (expr);                                                       \
    if (e_ != hipSuccess)                                                         \
      throw ::mfs::Error{MFS_EDEVICE, std::string(#expr) + ": " +                 \
                                          hipGetErrorString(e_)};                 \
  } while (0)

#define MFS_REQUIRE(cond, msg_expr)                                               \
  do {                                                                            \
    if (!(cond)) MFS_THROW(MFS_EINVAL, msg_expr);                                 \
  } while (0)

// --------------------------------------------------------- complex
__host__ __device__ inline double2 cz(double re, double im = 0.0) {
  double2 r;
  r.x = re;
  r.y = im;
  return r;
}
__host__ __device__ inline double2 cadd(double2 a, double2 b) { return cz(a.x + b.x, a.y + b.y); }
__host__ __device__ inline double2 csub(double2 a, double2 b) { return cz(a.x - b.x, a.y - b.y); }
__host__ __device__ inline double2 cmul(double2 a, double2 b) {
  return cz(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// conj(a) * b
__host__ __device__ inline double2 cmulc(double2 a, double2 b) {
  return cz(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__host__ __device__ inline double2 cscale(double2 a, double s) { return cz(a.x * s, a.y * s); }
__host__ __device__ inline double2 cconj(double2 a) { return cz(a.x, -a.y); }
__host__ __device__ inline double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }
// acc += a * b
__host__ __device__ inline void cfma(double2 &acc, double2 a, double2 b) {
  acc.x = fma(a.x, b.x, fma(-a.y, b.y, acc.x));
  acc.y = fma(a.x, b.y, fma(a.y, b.x, acc.y));
}
// acc += conj(a) * b
__host__ __device__ inline void cfmac(double2 &acc, double2 a, double2 b) {
  acc.x = fma(a.x, b.x, fma(a.y, b.y, acc.x));
  acc.y = fma(a.x, b.y, fma(-a.y, b.x, acc.y));
}

// cond ? a : b component by component (a select of the whole struct can be
// lowered through private memory)
__host__ __device__ inline double2 csel(bool cond, double2 a, double2 b) {
  return cz(cond ? a.x : b.x, cond ? a.y : b.y);
}

// p[i] if ok, else 0.  The load itself is unconditional (index 0 when !ok,
// so p must point at valid memory) and its bits are masked, not selected, so
// that the compiler cannot move it under a branch: a run of these is issued
// back to back instead of one branch and one wait per element.
__device__ inline double2 ld_or0(const double2 *p, size_t i, bool ok) {
  const double2 v = p[ok ? i : 0];
  const long long m = ok ? -1LL : 0LL;
  return cz(__longlong_as_double(__double_as_longlong(v.x) & m),
            __longlong_as_double(__double_as_longlong(v.y) & m));
}

// ----------------------------------------------------- kernel values
// A constant in scalar registers: the third operand of a fused multiply-add
// there, where the compiler would keep it in vector registers and copy it.
__device__ inline double scalar_const(double v) {
  asm("" : "+s"(v));
  return v;
}

// sin and cos of x, |x| <= kPhaseMax: x - n pi/2 in two terms of pi/2, the first
// difference exact with a fused multiply-add (a multiple of 2^-52 below 1), what
// rounding the second leaves off carried along; Taylor polynomials to r^17 and
// r^16 on |r| <= pi/4 (remainders under 1e-19), and the quadrant.  The largest
// error over 2e7 arguments is 0.95e-16.  (The library's sincos serves every
// argument, with a reduction that takes 50 registers beside it.)
constexpr double kPhaseMax = 1e15;
__device__ inline void sincos_mid(double x, double *sn, double *cs) {
  const double n = rint(x * scalar_const(0.63661977236758134308));
  const double p2 = scalar_const(-6.12323399573676603587e-17);
  const double t = fma(n, scalar_const(-1.57079632679489655800), x);
  const double r = fma(n, p2, t);
  const double rl = fma(n, p2, t - r);
  const double r2 = r * r;
  double s = fma(r2, scalar_const(1.0 / 355687428096000.0), -1.0 / 1307674368000.0);
  s = fma(r2, s, scalar_const(1.0 / 6227020800.0));
  s = fma(r2, s, scalar_const(-1.0 / 39916800.0));
  s = fma(r2, s, scalar_const(1.0 / 362880.0));
  s = fma(r2, s, scalar_const(-1.0 / 5040.0));
  s = fma(r2, s, scalar_const(1.0 / 120.0));
  s = fma(r2, s, scalar_const(-1.0 / 6.0));
  s = r + fma(r * r2, s, rl);
  double c = fma(r2, scalar_const(1.0 / 20922789888000.0), -1.0 / 87178291200.0);
  c = fma(r2, c, scalar_const(1.0 / 479001600.0));
  c = fma(r2, c, scalar_const(-1.0 / 3628800.0));
  c = fma(r2, c, scalar_const(1.0 / 40320.0));
  c = fma(r2, c, scalar_const(-1.0 / 720.0));
  c = fma(r2, c, scalar_const(1.0 / 24.0));
  const double w = fma(-0.5, r2, 1.0);   // cos r = w + (the rest of 1 - r^2 / 2) + ...
  c = w + fma(r2 * r2, c, fma(-r, rl, fma(-0.5, r2, 1.0 - w)));
  const int q = (int)fma(floor(n * 0.25), -4.0, n);   // n mod 4
  const double a = (q & 1) ? c : s, b = (q & 1) ? s : c;
  *sn = __hiloint2double(__double2hiint(a) ^ (int)((unsigned)(q & 2) << 30), __double2loint(a));
  *cs = __hiloint2double(__double2hiint(b) ^ (int)((unsigned)((q + 1) & 2) << 30), __double2loint(b));
}

// R = sqrt(r2) and 1 / R of a squared distance: the hardware's estimate of
// 1 / R (good to 2^-23) with one cubic step, and R = r2 / R corrected to half
// an ulp (it becomes the phase k R)
__device__ inline double dist(double r2, double &inv) {
  const double y = __builtin_amdgcn_rsq(r2);
  const double e = fma(-r2 * y, y, 1.0);
  inv = fma(y * e, fma(e, 0.375, 0.5), y);
  const double r = r2 * inv;
  return fma(fma(-r, r, r2), 0.5 * inv, r);
}

// ----------------------------------------------------- FP64 matrix cores
// One v_mfma_f64_16x16x4f64: D = A B + C with A 16 x 4 (lane i + 16 k holds
// A[i][k]), B 4 x 16 (lane j + 16 k holds B[k][j]) and C, D 16 x 16 (lane
// j + 16 g holds D[g + 4 v][j] in its v-th element; checked on gfx950 with
// a one-instruction probe).  Every lane of the wave must be active.
typedef double dx4 __attribute__((ext_vector_type(4)));

__device__ inline dx4 mfma_f64(double a, double b, dx4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ----------------------------------------------------- reductions
// DPP lane move of a double (both 32-bit halves with the same pattern);
// lanes whose source is outside the pattern, or whose row is masked off,
// receive 0.
template <int CTRL, int ROW_MASK>
__device__ inline double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ inline double lane63(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), 63);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
// Sum over the 64 lanes of a wave, returned to every lane.  An inclusive
// scan inside each row of 16 lanes (row_shr 1, 2, 4, 8), then row_bcast 15
// (rows 1 and 3 add the last lane of the row before) and row_bcast 31 (rows
// 2 and 3 add lane 31) leave the total in lane 63.  All 64 lanes must be
// active.
// Column sums of a lane-distributed block: every lane holds v[0..NB) (its
// row's terms of NB columns); on return lane l holds in v[0] the sum over
// all 64 lanes of column l % NB.  Plain sums over the lane bits above
// log2(NB), then a butterfly over the others that halves the values a lane
// keeps at each stage (63 exchanges for 64 columns instead of 6 a column).
// The stages are template recursions so that every index is a constant
// (the array stays in registers).
template <int O, int NB>
__device__ inline void plain_stages(double2 (&v)[NB]) {
  if constexpr (O >= NB) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      v[j].x += __shfl_xor(v[j].x, O, 64);
      v[j].y += __shfl_xor(v[j].y, O, 64);
    }
    plain_stages<O / 2, NB>(v);
  }
}
template <int H, int NB>
__device__ inline void butterfly_stages(double2 (&v)[NB], int lane) {
  if constexpr (H >= 1) {
    const bool hi = (lane & H) != 0;
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const double2 send = hi ? v[j] : v[j + H], keep = hi ? v[j + H] : v[j];
      v[j] = cz(keep.x + __shfl_xor(send.x, H, 64), keep.y + __shfl_xor(send.y, H, 64));
    }
    butterfly_stages<H / 2, NB>(v, lane);
  }
}
template <int NB>
__device__ inline void lane_column_sums(double2 (&v)[NB], int lane) {
  plain_stages<32, NB>(v);
  butterfly_stages<NB / 2, NB>(v, lane);
}

// v_permlane32_swap / v_permlane16_swap and an add: the sums of a's two halves
// (rows 2 i, 2 i + 1 of 16 lanes) in the lower lanes, of b's in the upper
__device__ inline double swap32_add(double a, double b) {
  const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
__device__ inline double swap16_add(double a, double b) {
  const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
// lane l's value (l uniform) to all lanes
__device__ inline double lane_value(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l), hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}
// the largest value of the wave, in every lane
__device__ inline double wave_max_dpp(double v) {
  v = fmax(v, dpp_move<0xb1, 0xf>(v));
  v = fmax(v, dpp_move<0x4e, 0xf>(v));
  v = fmax(v, dpp_move<0x141, 0xf>(v));
  v = fmax(v, dpp_move<0x140, 0xf>(v));
  {
    const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = fmax(__hiloint2double(h[0], l[0]), __hiloint2double(h[1], l[1]));
  }
  const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return fmax(__hiloint2double(h[0], l[0]), __hiloint2double(h[1], l[1]));
}

// lane C of every row of 16 lanes to the whole row (all lanes active)
template <int C>
__device__ inline double row_lane(double v) {
  return __longlong_as_double(
      __builtin_amdgcn_update_dpp(0L, (long)__double_as_longlong(v), 0x150 + C, 0xf, 0xf, true));
}
template <int C>
__device__ inline double2 row_lane(double2 v) {
  return cz(row_lane<C>(v.x), row_lane<C>(v.y));
}
// 16 x 16 matrices in a wave: lane c + 16 k holds the entries (4 u + k, c),
// u < 4, which is also the matrix cores' layout of A^T, B and D; a row goes to
// all lanes by lane swaps, a column by DPP.

// rows 4 u + KK, the lanes 16 KK .. 16 KK + 15, to all four rows of lanes
template <int KK>
__device__ inline double all_rows(double v) {
  const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  const auto l2 = __builtin_amdgcn_permlane16_swap(l[KK >> 1], l[KK >> 1], false, false);
  const auto h2 = __builtin_amdgcn_permlane16_swap(h[KK >> 1], h[KK >> 1], false, false);
  return __hiloint2double(h2[KK & 1], l2[KK & 1]);
}
template <int KK>
__device__ inline double2 all_rows(double2 v) {
  return cz(all_rows<KK>(v.x), all_rows<KK>(v.y));
}

// t <- t Y^{-1}, Y upper triangular, yinv the reciprocal of column c's diagonal entry
template <int P>
__device__ inline void rsolve16(double2 (&t)[4], const double2 (&y)[4], double2 yinv, int c) {
  if constexpr (P < 16) {
    const double2 yr = all_rows<P % 4>(y[P / 4]), yi = row_lane<P>(yinv);
    const double2 my = csel(c > P, cz(-yr.x, -yr.y), cz(0.0, 0.0));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double2 x = cmul(row_lane<P>(t[u]), yi);
      cfma(t[u], x, my);
      t[u] = csel(c == P, x, t[u]);
    }
    rsolve16<P + 1>(t, y, yinv, c);
  }
}

// re + i im += A B on the matrix cores: A (i, m) given as lane i + 16 k's entries
// m = 4 u + k, the others as above
__device__ inline void mfma16(const double2 (&a)[4], const double2 (&b)[4], dx4 &re, dx4 &im) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    re = mfma_f64(a[u].x, b[u].x, re);
    re = mfma_f64(-a[u].y, b[u].y, re);
    im = mfma_f64(a[u].x, b[u].y, im);
    im = mfma_f64(a[u].y, b[u].x, im);
  }
}
__device__ inline void mul16(const double2 (&a)[4], const double2 (&b)[4], double2 (&d)[4]) {
  dx4 re = {0, 0, 0, 0}, im = re;
  mfma16(a, b, re, im);
#pragma unroll
  for (int u = 0; u < 4; ++u) d[u] = cz(re[u], im[u]);
}

constexpr int QHR = 128;   // rows a workgroup in the reflector apply

__device__ inline double wave_sum(double v) {
  v += dpp_move<0x111, 0xf>(v);
  v += dpp_move<0x112, 0xf>(v);
  v += dpp_move<0x114, 0xf>(v);
  v += dpp_move<0x118, 0xf>(v);
  v += dpp_move<0x142, 0xa>(v);
  v += dpp_move<0x143, 0xc>(v);
  return lane63(v);
}
__device__ inline double2 wave_sum(double2 v) {
  v.x = wave_sum(v.x);
  v.y = wave_sum(v.y);
  return v;
}
__device__ inline double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }
inline int round_up(int a, int b) { return cdiv(a, b) * b; }

constexpr double kPi = 3.14159265358979323846;

}  // namespace mfs
