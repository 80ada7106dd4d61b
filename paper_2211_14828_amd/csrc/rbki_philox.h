// Counter-based Gaussian stream for the sketch matrix Omega (Alg. 1, step 1).
//
// Philox4x32-10 as published by Salmon, Moraes, Dror and Shaw ("Parallel
// random numbers: as easy as 1, 2, 3", SC'11): four 32-bit counter words,
// two key words, ten rounds.  One round multiplies c0 by 0xD2511F53 and c2 by
// 0xCD9E8D57 (64-bit products split into hi/lo halves) and maps
//   (c0, c1, c2, c3) -> (hi(c2*M1) ^ c1 ^ k0, lo(c2*M1), hi(c0*M0) ^ c3 ^ k1, lo(c0*M0));
// the key advances by (0x9E3779B9, 0xBB67AE85) between rounds.
//
// Gaussians by the Box-Muller transform (Box and Muller, 1958).  Stream
// conventions (seed, mode, tag, index) -> value:
//   key      = (seed mod 2^32, seed >> 32)
//   counter  = (lo32(L >> 1), hi32(L >> 1), mode, tag) for linear index L
//   u1, u2   = ((w0 * 2^20 + (w1 >> 12)) + 1/2) * 2^-52 and likewise (w2, w3)
//   z(L)     = sqrt(-2 ln u1) * (cos(2 pi u2) for even L, sin(2 pi u2) for odd L)
// Omega^(n)[j, s] is z at L = s * J_n + j with mode = n and tag = 0; so the
// buffer Omega^T (S x J, row-major) is the stream itself, in order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rbki {

struct PhiloxOut { uint32_t w0, w1, w2, w3; };

__host__ __device__ inline void mulhilo32(uint32_t a, uint32_t b, uint32_t& hi, uint32_t& lo) {
  uint64_t p = (uint64_t)a * (uint64_t)b;
  hi = (uint32_t)(p >> 32);
  lo = (uint32_t)p;
}

__device__ inline PhiloxOut philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                   uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    uint32_t hi0, lo0, hi1, lo1;
    mulhilo32(0xD2511F53u, c0, hi0, lo0);
    mulhilo32(0xCD9E8D57u, c2, hi1, lo1);
    uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);   // a ^ b ^ c
    uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  PhiloxOut o = {c0, c1, c2, c3};
  return o;
}

// 52-bit uniform in the open interval (0, 1); exact in double.
__host__ __device__ inline double unit_open(uint32_t wa, uint32_t wb) {
  return ((double)wa * 1048576.0 + (double)(wb >> 12) + 0.5) * 2.220446049250313080847e-16;  // 2^-52
}

// The Box-Muller pair (z(2m), z(2m+1)) for pair index m, in double.
__device__ inline void gauss_pair_f64(uint64_t m, uint32_t mode, uint32_t tag, uint64_t seed,
                                      double& z_even, double& z_odd) {
  PhiloxOut o = philox4x32_10((uint32_t)m, (uint32_t)(m >> 32), mode, tag, (uint32_t)seed,
                              (uint32_t)(seed >> 32));
  double u1 = unit_open(o.w0, o.w1);
  double u2 = unit_open(o.w2, o.w3);
  double r = sqrt(-2.0 * log(u1));
  double s, c;
  sincospi(2.0 * u2, &s, &c);
  z_even = r * c;
  z_odd = r * s;
}

// -ln u for u in (0, 1) (exact in double), in float to about an ulp.  u = 2^e (1 + f)
// with 1 + f in [sqrt(1/2), sqrt 2) and f taken in double, so that no accuracy goes
// as u nears 1; with s = f / (2 + f), ln(1 + f) = 2 atanh s
//   = f - (f^2/2 - s (f^2/2 + 2/3 s^2 + 2/5 s^4 + 2/7 s^6 + 2/9 s^8 + ...)),
// the next term below 2^-28 (s^2 <= 0.0295).
__device__ inline float minus_ln(double u) {
  int e = __builtin_amdgcn_frexp_exp(u);
  double m = __builtin_amdgcn_frexp_mant(u);          // [1/2, 1)
  const bool low = m < 0.70710678118654752;
  m = low ? 2.0 * m : m;
  e = low ? e - 1 : e;
  const float f = (float)(m - 1.0);
  const float h = 0.5f * f * f;
  const float s = f * __builtin_amdgcn_rcpf(2.0f + f);
  const float z = s * s;
  const float R = z * fmaf(z, fmaf(z, fmaf(z, 2.0f / 9.0f, 2.0f / 7.0f), 2.0f / 5.0f), 2.0f / 3.0f);
  // ln 2 in two parts, the first of 16 bits, so that its multiples are exact
  constexpr float LN2_HI = 0x1.62e4p-1f, LN2_LO = (float)(0.69314718055994530942 - 0x1.62e4p-1);
  const float k = (float)e;
  return -fmaf(k, LN2_HI, f - (h - fmaf(s, h + R, k * LN2_LO)));
}

// Same pair in single precision, for the float sketch.  The
// uniforms are exact in double, and so are the reductions of the logarithm's
// argument (above) and of the angle, 2 pi u2 = pi/2 (q + y) with q = round(4 u2), so
// the float arguments carry small absolute errors.  sin and cos of pi/2 y, |y| <=
// 1/2, by their power series to y^9 and y^10 (the next terms below 2^-28); the root
// by the hardware reciprocal root and one Newton step.  Against the library's log,
// log1p, sqrt and sincospi: 369 M values 0.96 -> 0.59 ms, the error against the
// double stream 5.5e-8 -> 4.5e-8 (root mean square), 8.5e-7 -> 6.7e-7 (largest).
__device__ inline void gauss_pair_f32(uint64_t m, uint32_t mode, uint32_t tag, uint64_t seed,
                                      float& z_even, float& z_odd) {
  PhiloxOut o = philox4x32_10((uint32_t)m, (uint32_t)(m >> 32), mode, tag, (uint32_t)seed,
                              (uint32_t)(seed >> 32));
  const float x = 2.0f * minus_ln(unit_open(o.w0, o.w1));
  const float rs = __builtin_amdgcn_rsqf(x), r0 = x * rs;
  const float r = fmaf(0.5f * fmaf(-r0, r0, x), rs, r0);
  const double t = 4.0 * unit_open(o.w2, o.w3);
  const double q = rint(t);                   // 0 .. 4
  const int qi = (int)q;
  const float y = (float)(t - q), w = y * y;
  // pi/2 (c - float(c)) joins the series' next term
  constexpr double H = 1.57079632679489661923, H2 = H * H, H3 = H2 * H, H5 = H3 * H2, H7 = H5 * H2, H9 = H7 * H2;
  constexpr float S0 = (float)H, S0L = (float)(H - (double)(float)H);
  constexpr float S1 = (float)(-H3 / 6), S2 = (float)(H5 / 120), S3 = (float)(-H7 / 5040), S4 = (float)(H9 / 362880);
  constexpr float C1 = (float)(-H2 / 2), C2 = (float)(H2 * H2 / 24), C3 = (float)(-H2 * H2 * H2 / 720),
                  C4 = (float)(H2 * H2 * H2 * H2 / 40320), C5 = (float)(-H2 * H2 * H2 * H2 * H2 / 3628800);
  const float sn = fmaf(y, S0, y * fmaf(w, fmaf(w, fmaf(w, fmaf(w, S4, S3), S2), S1), S0L));
  const float cs = fmaf(w, fmaf(w, fmaf(w, fmaf(w, fmaf(w, C5, C4), C3), C2), C1), 1.0f);
  const float a = qi & 1 ? sn : cs, b = qi & 1 ? cs : sn;
  const float c = ((qi + 1) & 2) ? -a : a, d = (qi & 2) ? -b : b;
  z_even = r * c;
  z_odd = r * d;
}

// The same pair for the bfloat16 sketches, whose values are rounded to bfloat16: the
// logarithm, root and sine and cosine of the library, with the same reductions in
// double (ln u1 as log1p(-(1 - u1)) when u1 >= 1/2; the angle 2 pi u2 as pi (x - n)
// with n = round(2 u2)).  It differs from the pair above in the last bits, and a value
// near a rounding edge of bfloat16 then moves by a whole step of 2^-8: that changes a
// basis of few steps by up to 1e-6, a factor's entries across their own edges in the
// first bfloat16 product, and so the core by some 1e-5.  The bfloat16 sketch of a seed
// is therefore fixed by this function.
__device__ inline void gauss_pair_bf16(uint64_t m, uint32_t mode, uint32_t tag, uint64_t seed,
                                       float& z_even, float& z_odd) {
  PhiloxOut o = philox4x32_10((uint32_t)m, (uint32_t)(m >> 32), mode, tag, (uint32_t)seed,
                              (uint32_t)(seed >> 32));
  const double u1 = unit_open(o.w0, o.w1);
  const double u2 = unit_open(o.w2, o.w3);
  const float ln = u1 < 0.5 ? logf((float)u1) : log1pf(-(float)(1.0 - u1));
  const float r = sqrtf(-2.0f * ln);
  const double x = 2.0 * u2;                  // angle / pi in (0, 2)
  const double nr = rint(x);                  // 0, 1 or 2
  float s, c;
  sincospif((float)(x - nr), &s, &c);
  if (nr == 1.0) { s = -s; c = -c; }          // shift by pi
  z_even = r * c;
  z_odd = r * s;
}

// The same pair for the block-scaled e4m3 sketch, whose values are rounded to
// bfloat16 and then to 3-bit mantissas under a shared power-of-two scale:
// uniforms from the first word of each half (u = (w + 1/2) 2^-32, in float),
// the hardware base-2 logarithm, square root, and sine and cosine of an
// argument in turns (sin(2 pi a)).  The values follow the stream above to
// about 1e-6, far below the bfloat16 step of 2^-8.
__device__ inline void gauss_pair_e4m3(uint64_t m, uint32_t mode, uint32_t tag, uint64_t seed,
                                       float& z_even, float& z_odd) {
  PhiloxOut o = philox4x32_10((uint32_t)m, (uint32_t)(m >> 32), mode, tag, (uint32_t)seed,
                              (uint32_t)(seed >> 32));
  const float u1 = fmaf((float)o.w0, 0x1p-32f, 0x1p-33f);
  const float a = fmaf((float)o.w2, 0x1p-32f, 0x1p-33f);
  const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));   // -2 ln 2 log2 u1
  z_even = r * __builtin_amdgcn_cosf(a);
  z_odd = r * __builtin_amdgcn_sinf(a);
}

}  // namespace rbki
