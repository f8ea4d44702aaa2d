// Twiddle-table description and the float64 evaluation of W_M^e shared by the
// host generator and the GPU generator, so both produce the same table.
//
// Sec. 2.3.1 precomputes sin and cos "by a certain angle" into a look-up
// table.  Here every table entry is W_M^e = exp(-2*pi*i*e/M) evaluated in
// float64 and rounded to float32.  The angle is reduced exactly with integer
// arithmetic first (eq. 3 periodicity, then quadrant and octant symmetry), so
// sin/cos only ever see an argument in [0, pi/4] and each entry is the float32
// nearest the true value except in vanishingly rare near-tie cases (and for two
// values in the stage tables, `balanced` below).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace mfft {

// Segment of a table: entries table[off + i], i < count, hold W_M^{e(i)} with
//   e(i) = (i / R) * (i % R) * mul   if R > 0  (2-D table: row i / R, column i % R)
//   e(i) = i * mul                   if R == 0 (linear table)
// or, with `rest`, what their rounding to float32 left out of them.
// `balanced` (stage tables and their larger factors): components of size cos(pi/16) and cos(pi/8) take
// the float32 above.  Those are the entries that repeat most, in every stage,
// and sqrt(1/2), cos(pi/8), cos(pi/16) all round down by 1.7e-8 to 3e-8 of
// their size: in one direction, such errors add up over the stages where others
// average out.  With two of them rounded up they cancel: 128 points as 2 x 8 x 8
// 8.94e-8 -> 8.69e-8 of the result (rms against 64 bits), 256 as 4 x 8 x 8
// 9.58e-8 -> 9.35e-8, 1024 as 4 x 16 x 16 1.091e-7 -> 1.064e-7, and with the
// same two constants in the 32-point butterfly 1024 as 32 x 32 1.113e-7 -> 1.064e-7.
struct TwSeg {
  int64_t off, count, R, M, mul;
  bool rest, balanced;
};
constexpr float kCosPi16Up = 0x1.f6297ep-1f, kCosPi8Up = 0x1.d906bep-1f;

__host__ __device__ inline int64_t seg_exponent(const TwSeg& s, int64_t i) {
  return s.R > 0 ? (i / s.R) * (i % s.R) * s.mul : i * s.mul;
}

// cos and sin of 2*pi*e/M in float64 (M a power of two, any integer e).
__host__ __device__ inline void twiddle_fp64(int64_t e, int64_t M, double* c_out, double* s_out) {
  const double half_pi = 1.57079632679489661923132169163975144;
  int64_t r = e % M;
  if (r < 0) r += M;
  // 2*pi*r/M = q*(pi/2) + (pi/2)*(rem/M), with rem = 4r - qM in [0, M)
  const int64_t q = (4 * r) / M;
  const int64_t rem = 4 * r - q * M;
  double cs, sn;
  if (2 * rem <= M) {
    const double a = half_pi * ((double)rem / (double)M);  // in [0, pi/4]
    cs = cos(a);
    sn = sin(a);
  } else {
    const double b = half_pi * ((double)(M - rem) / (double)M);  // in (0, pi/4)
    cs = sin(b);
    sn = cos(b);
  }
  switch (q & 3) {
    case 0: *c_out = cs; *s_out = sn; break;
    case 1: *c_out = -sn; *s_out = cs; break;
    case 2: *c_out = -cs; *s_out = -sn; break;
    default: *c_out = sn; *s_out = -cs; break;
  }
}

// The float32 of a balanced entry's component, and what its rounding left
// out: of a value rounded up a little less, so that the sum of the two still
// rounds to the value (half a step is 2.980e-8 there).
__host__ __device__ inline float round_balanced(double v, float* rest) {
  const double a = v < 0 ? -v : v;
  auto near = [a](double c) { return a - c < 1e-9 && c - a < 1e-9; };
  const float up = near(0.980785280403230449) ? kCosPi16Up : near(0.923879532511286756) ? kCosPi8Up : 0.0f;
  const float w = up > 0 ? up : (float)a, r = up > 0 ? -2.97e-8f : (float)(a - w);
  *rest = v < 0 ? -r : r;
  return v < 0 ? -w : w;
}

// Entry i of a segment.
__host__ __device__ inline float2 seg_value(const TwSeg& s, int64_t i) {
  double c, sn;
  twiddle_fp64(seg_exponent(s, i), s.M, &c, &sn);
  float2 w = make_float2((float)c, (float)-sn), rest = make_float2((float)(c - w.x), (float)(-sn - w.y));
  if (s.balanced) {
    w.x = round_balanced(c, &rest.x);
    w.y = round_balanced(-sn, &rest.y);
  }
  return s.rest ? rest : w;
}

hipError_t launch_twiddle_fp64(float2* table, const TwSeg* d_segs, int nseg, int64_t max_count,
                               hipStream_t s);

}  // namespace mfft
