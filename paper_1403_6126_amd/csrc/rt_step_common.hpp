// Device helpers of the two wave-group step kernels (rt_step3.hpp, FP32
// intensities; rt_step64.hpp, FP64): limiter, plane reads, reductions over the
// waves of a block, scalar angle records, and the reduced absorption system.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rt_common.hpp"
#include "rt_internal.hpp"

namespace rtk {

constexpr int kNsum = 22;        // per-cell sums of phase B
constexpr int kChunk = 11;       // values reduced per LDS round (22 sums, the moments)
constexpr int kRows = 13;        // folded sums, the values of the largest round

__device__ __forceinline__ double fma_(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}
// Half the van Leer harmonic-mean slope of two consecutive differences:
// ab/(a + b) when ab > 0, else 0 (zero at extrema).  The upwind interface
// value of the monotonic piecewise-linear reconstruction at Courant number
// nu is the upwind cell's value plus (1 - nu) times this, signed by the
// direction.  It is symmetric in a and b, odd under a, b -> -a, -b, exactly
// zero beside a zero difference (an empty cell has nothing to send out), and its
// rounding is relative to the slope.  The parabola (a + b) (phi - phi^2) of
// phi = b/(a + b), two instructions shorter, has none of this: its error is
// relative to the larger difference.
__device__ __forceinline__ double vl_half(double a, double b) {
  const double ab = a * b;
  const double q = ab * limiter_rcp(a + b);
  return ab > 0.0 ? q : 0.0;
}
// The multiplication whose product with zero is zero, whatever the other factor
// (the intrinsic by its name; the compiler has no builtin for it).
extern "C" __device__ __attribute__((const)) float fmul_legacy(float, float) __asm(
    "llvm.amdgcn.fmul.legacy");
// In FP32 the same value without the compare: max(ab, 0) times the reciprocal by
// the multiplication whose product with zero is zero (also where a + b = 0).
__device__ __forceinline__ float vl_half(float a, float b) {
  return fmul_legacy(fmaxf(a * b, 0.0f), limiter_rcp(a + b));
}

// Element idx of an angle plane, addressed by a 32-bit byte offset from the
// wave-uniform start of the plane (one scalar base and one vector register
// per load): planes of up to 4 GiB (plane_fits).
template <typename S>
__device__ __forceinline__ S plane_ld(const S *plane, unsigned idx) {
  const unsigned off = idx * (unsigned)sizeof(S);
  return *reinterpret_cast<const S *>(reinterpret_cast<const char *>(plane) + off);
}

// The same read as a raw buffer load: the plane is a buffer resource held in
// scalar registers, the lane's byte offset one vector register, so no vector
// address arithmetic is needed (gfx9 resource word 3 for raw loads).  The
// resource spans the whole 32-bit range: a read past its end returns zero.
template <typename S>
__device__ __forceinline__ S plane_buf_ld(const S *plane, unsigned idx) {
  const __amdgpu_buffer_rsrc_t r =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<S *>(plane), 0, -1, 0x00020000);
  const unsigned off = idx * (unsigned)sizeof(S);
  if constexpr (sizeof(S) == 8)
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  else
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// Sum (or, for the last value when MINLAST, minimum) of NV values over the
// G waves of the block, lane by lane, in a fixed order, R values per LDS
// round; every wave receives the totals.  The rounds only bound the LDS
// footprint (buf: G*R*64, tot: R*64 doubles): the result is the same for
// every R.
template <int NV, bool MINLAST, int R>
__device__ __forceinline__ void waves_reduce(double (&x)[NV], double *buf, double *tot, int g,
                                             int G, int lane) {
#pragma unroll
  for (int r0 = 0; r0 < NV; r0 += R) {
    const int nr = NV - r0 < R ? NV - r0 : R;
#pragma unroll
    for (int v = 0; v < R; ++v)
      if (v < nr) buf[(g * R + v) * 64 + lane] = x[r0 + v];
    __syncthreads();
    for (int v = g; v < nr; v += G) {
      double s = buf[v * 64 + lane];
      if (MINLAST && r0 + v == NV - 1) {  // wave-uniform branch
        for (int j = 1; j < G; ++j) {
          const double y = buf[(j * R + v) * 64 + lane];
          s = y < s ? y : s;
        }
      } else {
        for (int j = 1; j < G; ++j) s += buf[(j * R + v) * 64 + lane];
      }
      tot[v * 64 + lane] = s;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < R; ++v)
      if (v < nr) x[r0 + v] = tot[v * 64 + lane];
  }
}

// The new intensities and the per-cell outputs are written once and not read
// again by the step: with RT_STREAM_STORES they bypass the caches as
// non-temporal stores, leaving L2 to the stencil reuse and the spill.
#ifndef RT_STREAM_STORES
#define RT_STREAM_STORES 1
#endif
template <typename T>
__device__ __forceinline__ void stream_store(T *p, T v) {
  if constexpr (RT_STREAM_STORES)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// A pointer into the constant address space: the angle records are read-only
// for the whole step, and reads through such a pointer at a wave-uniform
// address become scalar loads even after the step's global writes and
// atomics (through a generic pointer the compiler makes vector loads of
// them there).  128^3 S8: FP64 3.56 -> 3.18 ms, FP32 1.79 -> 1.58 ms.
#ifndef RT_CONST_RECORDS
#define RT_CONST_RECORDS 1
#endif
#if RT_CONST_RECORDS
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;
#else
template <typename T>
using cptr = const T *;
#endif

// A zero that the compiler cannot see through, added to the address of the
// angle records at the start of a phase: what one phase loads is then not kept
// in (spilled) scalar registers for the next.
__device__ __forceinline__ int opaque_zero() {
  int z;
  asm volatile("s_mov_b32 %0, 0" : "=s"(z));
  return z;
}

// The record of angle m (StepArgs::arec) in the arithmetic type.
template <typename A>
__device__ __forceinline__ cptr<A> angle_rec(const StepArgs &p, int m) {
  if constexpr (sizeof(A) == 4)
    return (cptr<A>)(p.arecf + (size_t)m * kRec);
  else
    return (cptr<A>)(p.arec + (size_t)m * kRec);
}

// The reduced absorption system of one cell (Section 4.3, Eq.
// absorptionmatrix): from the angle sums S[0..8] (sum W r/D, W e/D, W/D,
// the same weighted by n.u and by u^2 + (n.u)^2) the temperature equation is
// one quartic, c_v (T' - T^n) = h0 + h1q T'^4, solved by Newton's method in
// FP64 from T^n; returns T' and sets X = T'^4/(4 pi), Q (the n.u-weighted
// intensity sum of the solution), the iteration count and convergence.
template <int NV>
__device__ __forceinline__ double absorb_solve(const StepArgs &p, const double (&S)[NV], double kap,
                                               double uu, double cv, double Tn, double sa,
                                               double &X, double &Q, int &it, bool &conv) {
  const double C = p.C, P = p.P, dt = p.dt, iC = p.invC;
  const double qden = 1.0 + kap * S[8];
  const double iqden = fast_rcp(qden);
  const double q0 = S[6] * iqden, q1 = S[7] * iqden;
  const double j0 = S[0] - kap * S[2] * q0, j1 = S[1] - kap * S[2] * q1;
  const double k0 = S[3] - kap * S[5] * q0, k1 = S[4] - kap * S[5] * q1;
  const double beta = P * C * (1.0 - uu * iC * iC) * sa * dt;
  const double g8 = 8.0 * kPi * P * sa * dt;
  const double h0 = -g8 * (k0 - q0 * iC) + kFourPi * beta * j0;
  const double h1q = (-g8 * (k1 - q1 * iC) - kFourPi * beta * (1.0 - j1)) * (1.0 / kFourPi);
  double T = Tn;
  conv = false;
  for (it = 1; it <= p.maxit; ++it) {
    const double T3 = T * T * T;
    const double f = cv * (T - Tn) - h0 - h1q * T3 * T;
    const double dT = f * fast_rcp(cv - 4.0 * h1q * T3);
    T -= dT;
    if (fabs(dT) <= p.rtol * fabs(T)) {
      conv = true;
      break;
    }
  }
  X = T * T * T * T * (1.0 / kFourPi);
  Q = q0 + q1 * X;
  return T;
}

// The 22 angle sums of the reduced absorption and scattering systems at one
// velocity u from 13.  With t = n.u, D = D0 - a t and w = AW0 - s t (the
// diagonals; a = dt sigma_a, s = dt sigma_s), every sum that does not hold an
// intensity is a combination of A_k = sum W t^k/D, B_k = sum W t^k/w and
// C_k = sum W t^k/(w D), k = 0..3, and those follow downwards from k = 3:
//   D0 A_k = M_k + a A_{k+1},  AW0 B_k = M_k + s B_{k+1},  D0 C_k = B_k + a C_{k+1},
// with the moments M_k = sum W t^k (k = 0..2) of the angle set contracted with
// u.  The sums with the right-hand side r follow the same way from
// R_2 = sum W t^2 r/D and the moments of r, those with p = r/D + g5 dF from
// P_2 = sum W t^2 p/w and the moments of r and g5 dF.  All terms added are of
// one size or falling with |u|/C, so nothing cancels.
//   f[0..3] sum W r, W n r; f[4..7] the same of g5 dF; f[8] R_2; f[9] P_2;
//   f[10..12] A_3, B_3, C_3.  wm: sum W, W n_i, W n_i n_j (xx yy zz xy xz yz).
// Fills S[0..10] and Q[0..7] (sums 11..18).
__device__ __forceinline__ void unfold_sums(const double (&f)[13], const double (&wm)[10],
                                            double u0, double u1, double u2, double uu, double D0,
                                            double a, double E0, double AW0, double s, double B0,
                                            double sC, double (&S)[11], double (&Q)[11]) {
  const double iD0 = fast_rcp(D0), iAW = fast_rcp(AW0);
  const double m0 = wm[0], m1 = u0 * wm[1] + u1 * wm[2] + u2 * wm[3];
  const double m2 = u0 * (u0 * wm[4] + 2.0 * (u1 * wm[7] + u2 * wm[8])) +
                    u1 * (u1 * wm[5] + 2.0 * u2 * wm[9]) + u2 * u2 * wm[6];
  const double A3 = f[10], A2 = (m2 + a * A3) * iD0, A1 = (m1 + a * A2) * iD0,
               A0 = (m0 + a * A1) * iD0;
  const double B3 = f[11], B2 = (m2 + s * B3) * iAW, B1 = (m1 + s * B2) * iAW,
               Bz = (m0 + s * B1) * iAW;
  const double C3 = f[12], C2 = (B2 + a * C3) * iD0, C1 = (B1 + a * C2) * iD0,
               C0 = (Bz + a * C1) * iD0;
  const double R2 = f[8], R1 = (u0 * f[1] + u1 * f[2] + u2 * f[3] + a * R2) * iD0,
               R0 = (f[0] + a * R1) * iD0;
  const double P2 = f[9], P1 = (R1 + (u0 * f[5] + u1 * f[6] + u2 * f[7]) + s * P2) * iAW,
               P0 = (R0 + f[4] + s * P1) * iAW;
  const double a3 = 3.0 * a, s2 = 2.0 * s, s3 = -3.0 * s;
  S[0] = R0;                              // W r/D
  S[1] = E0 * A0 + a3 * A1;               // W e/D
  S[2] = A0;                              // W/D
  S[3] = R1;                              // W t r/D
  S[4] = E0 * A1 + a3 * A2;               // W t e/D
  S[5] = A1;                              // W t/D
  S[6] = uu * R0 + R2;                    // W g r/D
  S[7] = uu * S[1] + E0 * A2 + a3 * A3;   // W g e/D
  S[8] = uu * A0 + A2;                    // W g/D
  S[9] = B0 * P0 + s2 * P1 - sC * P2;     // W b p/w
  S[10] = P0;                             // W p/w
  Q[0] = B0 * Bz + s2 * B1 - sC * B2;     // W b/w
  Q[1] = s3 * (B0 * B1 + s2 * B2 - sC * B3);  // W b c/w
  Q[2] = Bz;                              // W/w
  Q[3] = s3 * B1;                         // W c/w
  const double b0 = B0 * C0 + s2 * C1 - sC * C2, b1 = B0 * C1 + s2 * C2 - sC * C3;
  Q[4] = E0 * b0 + a3 * b1;               // W b e/(w D)
  Q[5] = b0;                              // W b/(w D)
  Q[6] = E0 * C0 + a3 * C1;               // W e/(w D)
  Q[7] = C0;                              // W/(w D)
}

}  // namespace rtk
