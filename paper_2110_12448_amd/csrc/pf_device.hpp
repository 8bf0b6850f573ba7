// pf_device.hpp -- device-side building blocks shared by the gfx950 step and
// reduction kernels: per-precision math, wave64 cross-lane moves, boundary
// ghost maps and buffer stores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pf_internal.hpp"

namespace pf {

// ------------------------------------------------------------------ math

template <typename T> struct Math;

template <> struct Math<float> {
  static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
  static __device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
  // tanh(x) = sign(x) (1 - e) / (1 + e), e = exp(-2|x|), with the hardware
  // base-2 exponential; absolute error a few ulp of 1.
  static __device__ __forceinline__ float tanh_(float x) {
    const float m2log2e = -2.8853900817779268f;  // -2 / ln 2
    float e = __builtin_amdgcn_exp2f(m2log2e * __builtin_fabsf(x));
    float t = (1.0f - e) * __builtin_amdgcn_rcpf(1.0f + e);
    return __builtin_copysignf(t, x);
  }
  // phi = tanh(psi / sqrt2) = sign(psi) (1 - e) / (1 + e), e = exp(-sqrt2
  // |psi|), with the hardware base-2 exponential; absolute error a few ulp of 1.
  static __device__ __forceinline__ float phi(float psi) {
    const float c = -2.0402789f;  // -sqrt2 / ln 2
    const float e = __builtin_amdgcn_exp2f(c * __builtin_fabsf(psi));
    return __builtin_copysignf((1.0f - e) * __builtin_amdgcn_rcpf(1.0f + e), psi);
  }
  static __device__ __forceinline__ bool finite(float x) { return __builtin_isfinite(x); }
};

// FP64: the hardware seeds (about 2^-24) and one third-order Newton step in
// place of the IEEE division and square-root sequences, and a tanh of its own.
// The arguments are finite, those of rsq positive; a zero gives NaN (inf in
// FP32), which callers select away (the gradients of uniform cells).
// Against 80-bit results over 2M arguments: rcp max 0.500 ulp, rms 0.289 (x/y
// 0.500 and 0.289); rsq 0.99 and 0.34 (1/sqrt 1.48 and 0.46); tanh 0.86 and
// 0.29 (the runtime library's 0.86 and 0.28).
template <> struct Math<double> {
  static __device__ __forceinline__ double rcp(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, __builtin_fma(e, e, e), r);
  }
  static __device__ __forceinline__ double rsq(double x) {
    const double r = __builtin_amdgcn_rsq(x);
    const double e = __builtin_fma(-(x * r), r, 1.0);
    return __builtin_fma(r * e, __builtin_fma(0.375, e, 0.5), r);
  }
  // tanh(x) = sign(x) * -E / (2 + E), E = expm1(-2|x|): Cody-Waite reduction
  // y = n ln2 + r, expm1(r) = r + r^2 (1/2 + r g(r)) with g from Chebyshev
  // interpolation on |r| <= ln2 / 2 (error 8e-18), E = 2^n expm1(r) + (2^n - 1)
  // and the quotient in head and tail parts.
  static __device__ __forceinline__ double tanh_(double x) {
    const double kLog2e = 0x1.71547652b82fep+0, kLn2Hi = 0x1.62e42fee00000p-1,
                 kLn2Lo = 0x1.a39ef35793c76p-33, kMagic = 6755399441055744.0;  // 1.5 * 2^52
    double ax = __builtin_fabs(x);
    ax = ax > 40.0 ? 40.0 : ax;  // 1 from 19.1 on; a NaN stays
    const double y = -2.0 * ax;
    const double t = __builtin_fma(y, kLog2e, kMagic);
    const double n = t - kMagic;
    const int ni = (int)__builtin_bit_cast(unsigned long long, t);
    const double r1 = __builtin_fma(n, -kLn2Hi, y);
    const double r = __builtin_fma(n, -kLn2Lo, r1);
    const double rl = __builtin_fma(n, -kLn2Lo, r1 - r);
    double g = 0x1.1f66f85dfa20ap-29;
    g = __builtin_fma(g, r, 0x1.af38d53857513p-26);
    g = __builtin_fma(g, r, 0x1.27e4e1ea0f53ap-22);
    g = __builtin_fma(g, r, 0x1.71de0d9c145d0p-19);
    g = __builtin_fma(g, r, 0x1.a01a01a47db6fp-16);
    g = __builtin_fma(g, r, 0x1.a01a01a7c8d47p-13);
    g = __builtin_fma(g, r, 0x1.6c16c16c167dep-10);
    g = __builtin_fma(g, r, 0x1.11111111109adp-7);
    g = __builtin_fma(g, r, 0x1.5555555555555p-5);
    g = __builtin_fma(g, r, 0x1.5555555555556p-3);
    g = __builtin_fma(g, r, 0.5);
    const double c = __builtin_fma(r * r, g, rl);  // expm1(y - n ln2) = r + c
    const double s =  // 2^n
        __builtin_bit_cast(double, (unsigned long long)(unsigned)((ni << 20) + 0x3ff00000) << 32);
    const double a = s - 1.0, b = s * r, h0 = a + b;
    double lo = (b - (h0 - a)) + (s - (a + 1.0));
    lo = __builtin_fma(s, c, lo);
    const double hi = h0 + lo;
    lo = lo - (hi - h0);
    const double dh = 2.0 + hi, dl = (hi - (dh - 2.0)) + lo;
    const double q = rcp(dh), v = -hi * q;
    const double rem = __builtin_fma(-v, dl, __builtin_fma(-v, dh, -hi)) - lo;
    return __builtin_copysign(__builtin_fma(rem, q, v), x);
  }
  static __device__ __forceinline__ double phi(double psi) {
    return tanh_(psi * 0.70710678118654752);
  }
  static __device__ __forceinline__ bool finite(double x) { return __builtin_isfinite(x); }
};

// A wait state between vector instructions, tied to the value x so that it is
// issued where x is formed.  Two waves of a SIMD issue FP32 instructions on
// vector registers side by side (2.2 cycles each measured), but a lane move,
// a transcendental or a readlane leaves them issuing in turn (4.2), also if
// only one instruction in 50 is one, until one of the waves issues something
// else; a scalar instruction every 4 to 12 vector ones restores the pairing
// (a mix like the step's: 4.2 -> 3.1 cycles an instruction at 4 waves per
// SIMD, 4.5 -> 3.3 at 2).  FP64 instructions do not pair.
template <bool kOn = true, typename T>
__device__ __forceinline__ void pause_issue(T &x) {
  if constexpr (kOn && sizeof(T) == 4) asm("s_nop 0" : "+v"(x));
}

// ------------------------------------------------------- frame decision
// A phi = 0 crossing between rows m and m + 1 (phi_m >= 0 > phi_{m+1}) lies
// at height y = (m + phi_m / (phi_m - phi_{m+1})) h; the frame moves when some
// y >= shift_row h, both sides rounded in FP64 (thr = shift_row h).  The
// fraction lies in [0, 1], so a crossing from a row at or above shift_row
// always qualifies and one from a row below shift_row - 1 never does (FP64
// rounding is monotone and cannot close a gap of h): callers skip those rows
// and only the row just below shift_row evaluates the quotient.
template <typename T>
__device__ __forceinline__ bool crossing_reaches(T fC, T fN, int m, int shift_row, double thr,
                                                 double hd) {
  if (m >= shift_row) return true;
  const double fc = (double)fC, fn = (double)fN;
  return ((double)m + fc / (fc - fn)) * hd >= thr;
}

// ------------------------------------------------------- cross-lane moves
// Lane i of a wave64 holds lattice column x0 + i.  from_right() returns the
// value of lane i + 1 (column x + 1), from_left() the value of lane i - 1;
// the end lanes receive 0.  Both are single DPP wave shifts.

#define PF_DPP_WAVE_SHL1 0x130  // lane i reads lane i + 1
#define PF_DPP_WAVE_SHR1 0x138  // lane i reads lane i - 1

__device__ __forceinline__ float from_right(float v) {
  return __builtin_amdgcn_update_dpp(0.0f, v, PF_DPP_WAVE_SHL1, 0xF, 0xF, true);
}
__device__ __forceinline__ float from_left(float v) {
  return __builtin_amdgcn_update_dpp(0.0f, v, PF_DPP_WAVE_SHR1, 0xF, 0xF, true);
}
__device__ __forceinline__ double from_right(double v) {
  int2 a = __builtin_bit_cast(int2, v);
  a.x = __builtin_amdgcn_update_dpp(0, a.x, PF_DPP_WAVE_SHL1, 0xF, 0xF, true);
  a.y = __builtin_amdgcn_update_dpp(0, a.y, PF_DPP_WAVE_SHL1, 0xF, 0xF, true);
  return __builtin_bit_cast(double, a);
}
__device__ __forceinline__ double from_left(double v) {
  int2 a = __builtin_bit_cast(int2, v);
  a.x = __builtin_amdgcn_update_dpp(0, a.x, PF_DPP_WAVE_SHR1, 0xF, 0xF, true);
  a.y = __builtin_amdgcn_update_dpp(0, a.y, PF_DPP_WAVE_SHR1, 0xF, 0xF, true);
  return __builtin_bit_cast(double, a);
}
__device__ __forceinline__ int from_right(int v) {
  return __builtin_amdgcn_update_dpp(0, v, PF_DPP_WAVE_SHL1, 0xF, 0xF, true);
}
__device__ __forceinline__ int from_left(int v) {
  return __builtin_amdgcn_update_dpp(0, v, PF_DPP_WAVE_SHR1, 0xF, 0xF, true);
}

// ------------------------------------------------------------- ghost maps
// Lattice index i (possibly outside [0, n)) -> stored index.  PERIODIC wraps;
// NOFLUX mirrors about the boundary face (-1 -> 0, -2 -> 1, n -> n-1, ...).
__device__ __forceinline__ int ghost(int i, int n, int bc) {
  if (bc == PF_BC_PERIODIC) {
    int m = i % n;
    return m < 0 ? m + n : m;
  }
  int p = 2 * n;
  int m = i % p;
  if (m < 0) m += p;
  return m < n ? m : p - 1 - m;
}

// Same map for indices within one period of the lattice (-n <= i < 2n), with
// no division: used for row indices inside the time-step loops.
__device__ __forceinline__ int ghost_near(int i, int n, int bc) {
  if (i < 0) return bc == PF_BC_PERIODIC ? i + n : -i - 1;
  if (i >= n) return bc == PF_BC_PERIODIC ? i - n : 2 * n - 1 - i;
  return i;
}

// Store v at column x of the row starting at `row` (nx elements) from the
// lanes with ok set, without a branch: a raw buffer store whose record is the
// row, the other lanes given an offset beyond it, which the hardware drops.
// Straight-line stores keep the row pipelines of the step kernels in fewer
// basic blocks.
template <typename T>
__device__ __forceinline__ void store_row(T *row, int nx, int x, bool ok, T v) {
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(row, 0, nx * (int)sizeof(T), 0x00020000);  // word 3: raw 32-bit access (gfx9 family)
  // the dropped lanes' offset 2^31 lies past every record: nx * 8 < 2^31
  // because the x-y plane is at most 2^30 - 1 cells and ny >= 4
  const int off = ok ? x * (int)sizeof(T) : (int)0x80000000u;
  if constexpr (sizeof(T) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, off, 0, 0);
  } else {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), rs, off, 0, 0);
  }
}

}  // namespace pf
