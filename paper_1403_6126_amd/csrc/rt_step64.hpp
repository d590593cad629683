// FP64 step kernel: the waves of a block share 64 cells, each owns a run of
// angles, and faces between cells are formed once where a neighbour can pass
// them on.
//
// A block holds 64 consecutive cells, one per lane, and G waves; wave g owns
// the NS angles g NS .. g NS + NS - 1 (in chunks of G NS when the set is larger
// than that).  Within a wave the angle is uniform: direction cosines, weights
// and signs are scalars, and every intensity load reads 64 consecutive cells
// of one plane.  Per step of a tile:
//   build    the waves share the work that every angle needs: the face data of
//            each axis and the cell's velocity estimate, written to LDS;
//   phase A  transport increments (Section 4.2), axis by axis;
//   phase B  right-hand sides and 13 angle sums, reduced over the waves;
//   solve    the 22 sums of the reduced systems from the 13, FP64 Newton on the
//            quartic in T', the 2 x 2 scattering system (wave 0);
//   phase C  I^{n+1}, its moments, the gas source terms.
//
// What bounds it: instruction issue and the latency of the waves, not HBM
// (128^3 S8: 3.2 GB of algorithmic bytes, 0.7 ms at the rate of a large copy).
// Each of an axis's two faces costs two limiters with a reciprocal each and the IV
// differences, about 40 instructions.  Faces along x are therefore shared: a lane
// computes its high face and takes the low one from the lane below (a DPP wave
// shift); the low faces of the few lanes that have no such neighbour (lane 0 and
// the first cell of a row) are computed together, one lane per (angle, cell),
// before phase A.  The other axes form both faces in each cell.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rt_common.hpp"
#include "rt_internal.hpp"
#include "rt_step_common.hpp"

namespace rtk {

enum Mode64 : int { kFused64 = 0, kSource64 = 1 };

// Data of one face between the cells at offsets 0 and +1 along an axis.  With
// I~ = I - IV/C, D the difference of I~ over the face (upper minus lower),
// D_x that of the interval upwind of it, V and V_x those of IV, q and qv the
// half slopes of the upwind cells, the face value relative to the lower cell,
// in units of the increment, is
//   G = k D + sign(mu) h2 Ca q + r V + f qv,   k = Cb (mu > 0), Ca + Cb (mu < 0),
// with Ca = C alpha, Cb = C (1 - alpha)/2, h2 = 1 - nu, r the upper cell's
// share of the IV value and f its signed slope factor (all times dt/dx).
// Relative to the upper cell it is G - C dt/dx (I_+1 - I_0), since the value
// of I~ and that of IV add to I; as Ca + 2 Cb = C this is the same sum with
// k - C = -Cb - Ca (mu > 0), -Cb (mu < 0) in place of k and r - 1 = -l in place
// of r, which is how it is formed: a face beside an empty upwind cell is then
// zero exactly, relative to that cell.  The increment of a cell is -mu times
// the difference of its two faces relative to the cell.
struct Face64 {
  unsigned idx[4];  // cells at offsets -1, 0, +1, +2 (wrapped, or the edge cell)
  unsigned kinds;   // bit j: cell j is a ghost of a fixed or vacuum face
  double w0[3];     // W(+1) - W(0), W = 3 v J
  double wm[3];     // W(0) - W(-1): the interval below
  double wp[3];     // W(+2) - W(+1): the interval above
  double wf[3];     // wm or wp, the one upwind by the flow of the face
  double ca, cb, r, f;
  double l;         // dt/dx - r, the lower cell's share
};
constexpr int kFaceVals = 16, kFaceWords = 5;

// The cell at coordinate k along axis d (k = -2 .. n + 1), cb the cell at
// coordinate 0; kind: 1 where it is a ghost that does not copy the cell (fixed
// and vacuum faces).  at: where its intensities are read, the
// cell itself or, for a ghost with a fixed table, its place in a
// position-dependent one (face cells in order of the two other axes).
template <bool PER>
__device__ __forceinline__ unsigned stencil_cell(const StepArgs &p, int cb, int k, int d,
                                                 unsigned &at, unsigned &kind) {
  const int n = p.n[d];
  const bool below = k < 0, out = below || k >= n;
  const int bc = PER ? kPeriodic : p.bc[d][below ? 0 : 1];
  if (bc == kPeriodic) {  // at most two cells out: one wrap, two where n = 1
    k += k < 0 ? n : 0;
    k += k < 0 ? n : 0;
    k -= k >= n ? n : 0;
    k -= k >= n ? n : 0;
  } else {
    k = k < 0 ? 0 : k >= n ? n - 1 : k;
  }
  const unsigned c = (unsigned)(cb + k * p.stride[d]);
  at = c;
  kind = 0;
  if (!PER && out) {
    kind = bc == kFixed || bc == kVacuum ? 1u : 0u;
    if (bc == kFixed) {
      const unsigned n0 = (unsigned)p.n[0], n01 = n0 * (unsigned)p.n[1];
      at = d == 0 ? c / n0 : d == 1 ? c % n0 + n0 * (c / n01) : c % n01;
    }
  }
  return c;
}

// The coefficients of the face between coordinates k and k + 1 along axis d,
// lo and up its two cells (the edge cell at a boundary).
template <bool PER>
__device__ __forceinline__ void face_coef64(const StepArgs &p, unsigned lo, unsigned up, int k,
                                            int d, double &ca, double &cb, double &r, double &f) {
  const size_t N = (size_t)p.ncell;
  double l;
  if (PER || k + 1 < p.n[d] || p.bc[d][1] == kPeriodic) {
    // the low face of the cell above (at a low boundary, of the first cell)
    ca = p.faces[(size_t)(d * 3 + 0) * N + up];
    l = p.faces[(size_t)(d * 3 + 1) * N + up];
    f = p.faces[(size_t)(d * 3 + 2) * N + up];
  } else {
    // high non-periodic boundary: the ghost copies the edge cell's fields
    const double u = p.v[(size_t)d * N + lo];
    ca = p.C * alpha_of(p.sa[lo] + p.ss[lo], p.dl10[d]);
    l = iv_lower_share(u);
    f = iv_signed_factor(u, p.dt_dx[d]);
  }
  const double s = p.dt_dx[d];
  cb = (0.5 * p.C - 0.5 * ca) * s;
  ca *= s;
  r = (1.0 - l) * s;
  f *= s;
}

// The face between coordinates k and k + 1 along axis d (k = -1 .. n - 1).
template <bool PER>
__device__ __forceinline__ void load_face64(const StepArgs &p, int cb, int k, int d, Face64 &f) {
  const size_t N = (size_t)p.ncell;
  double W[4][3];
  unsigned cell[4];
  f.kinds = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    unsigned kind;
    cell[j] = stencil_cell<PER>(p, cb, k - 1 + j, d, f.idx[j], kind);
    f.kinds |= kind << j;
#pragma unroll
    for (int t = 0; t < 3; ++t) W[j][t] = p.mom_in[(size_t)(10 + t) * N + cell[j]];
  }
  face_coef64<PER>(p, cell[1], cell[2], k, d, f.ca, f.cb, f.r, f.f);
  f.l = p.dt_dx[d] - f.r;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    f.wm[t] = W[1][t] - W[0][t];
    f.w0[t] = W[2][t] - W[1][t];
    f.wp[t] = W[3][t] - W[2][t];
    f.wf[t] = f.f > 0.0 ? f.wm[t] : f.wp[t];
  }
}

// Rows of 64 lanes in LDS: kFaceVals doubles, then kFaceWords words.
constexpr size_t face_lds_bytes() { return 64 * (kFaceVals * 8 + kFaceWords * 4); }
__device__ __forceinline__ void face_put(char *b, const Face64 &f, int lane) {
  double *v = reinterpret_cast<double *>(b) + lane;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    v[t * 64] = f.w0[t];
    v[(3 + t) * 64] = f.wm[t];
    v[(6 + t) * 64] = f.wp[t];
    v[(9 + t) * 64] = f.wf[t];
  }
  v[12 * 64] = f.ca;
  v[13 * 64] = f.cb;
  v[14 * 64] = f.r;
  v[15 * 64] = f.f;
  unsigned *w = reinterpret_cast<unsigned *>(b + 64 * kFaceVals * 8) + lane;
#pragma unroll
  for (int j = 0; j < 4; ++j) w[j * 64] = f.idx[j];
  w[4 * 64] = f.kinds;
}
__device__ __forceinline__ void face_get(const char *b, double dt_dx, Face64 &f, int lane) {
  const double *v = reinterpret_cast<const double *>(b) + lane;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    f.w0[t] = v[t * 64];
    f.wm[t] = v[(3 + t) * 64];
    f.wp[t] = v[(6 + t) * 64];
    f.wf[t] = v[(9 + t) * 64];
  }
  f.ca = v[12 * 64];
  f.cb = v[13 * 64];
  f.r = v[14 * 64];
  f.l = dt_dx - f.r;
  f.f = v[15 * 64];
  const unsigned *w = reinterpret_cast<const unsigned *>(b + 64 * kFaceVals * 8) + lane;
#pragma unroll
  for (int j = 0; j < 4; ++j) f.idx[j] = w[j * 64];
  f.kinds = w[4 * 64];
}

// Data of a cell along an axis on which it forms both faces: cells -2, -1, +1,
// +2, the four W differences and the coefficients of the two faces.
struct Both64 {
  unsigned idx[4], kinds;
  double w[4][3];
  double caL, cbL, caR, cbR, lL, rR, fL, fR;
};
constexpr int kBothVals = 20, kBothWords = 5;
constexpr size_t both_lds_bytes() { return 64 * (kBothVals * 8 + kBothWords * 4); }

template <bool PER>
__device__ __forceinline__ void load_both64(const StepArgs &p, int c, int k, int d, Both64 &b) {
  const size_t N = (size_t)p.ncell;
  const int cb = c - k * p.stride[d];
  unsigned cell[4];
  b.kinds = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    unsigned kind;
    cell[j] = stencil_cell<PER>(p, cb, k + (j < 2 ? j - 2 : j - 1), d, b.idx[j], kind);
    b.kinds |= kind << j;
  }
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const double *W = p.mom_in + (size_t)(10 + t) * N;
    const double Wm = W[cell[1]], Wc = W[c], Wp = W[cell[2]];
    b.w[0][t] = Wm - W[cell[0]];
    b.w[1][t] = Wc - Wm;
    b.w[2][t] = Wp - Wc;
    b.w[3][t] = W[cell[3]] - Wp;
  }
  double rL;
  face_coef64<PER>(p, cell[1], (unsigned)c, k - 1, d, b.caL, b.cbL, rL, b.fL);
  b.lL = p.dt_dx[d] - rL;  // the lower cell's share
  face_coef64<PER>(p, (unsigned)c, cell[2], k, d, b.caR, b.cbR, b.rR, b.fR);
}
__device__ __forceinline__ void both_put(char *m, const Both64 &b, int lane) {
  double *v = reinterpret_cast<double *>(m) + lane;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int t = 0; t < 3; ++t) v[(j * 3 + t) * 64] = b.w[j][t];
  const double co[8] = {b.caL, b.cbL, b.caR, b.cbR, b.lL, b.rR, b.fL, b.fR};
#pragma unroll
  for (int j = 0; j < 8; ++j) v[(12 + j) * 64] = co[j];
  unsigned *w = reinterpret_cast<unsigned *>(m + 64 * kBothVals * 8) + lane;
#pragma unroll
  for (int j = 0; j < 4; ++j) w[j * 64] = b.idx[j];
  w[4 * 64] = b.kinds;
}
__device__ __forceinline__ void both_get(const char *m, Both64 &b, int lane) {
  const double *v = reinterpret_cast<const double *>(m) + lane;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int t = 0; t < 3; ++t) b.w[j][t] = v[(j * 3 + t) * 64];
  b.caL = v[12 * 64];
  b.cbL = v[13 * 64];
  b.caR = v[14 * 64];
  b.cbR = v[15 * 64];
  b.lL = v[16 * 64];
  b.rR = v[17 * 64];
  b.fL = v[18 * 64];
  b.fR = v[19 * 64];
  const unsigned *w = reinterpret_cast<const unsigned *>(m + 64 * kBothVals * 8) + lane;
#pragma unroll
  for (int j = 0; j < 4; ++j) b.idx[j] = w[j * 64];
  b.kinds = w[4 * 64];
}

// The ghost intensity of angle m beyond face (d, side): the fixed table's (at
// as in stencil_cell, read only where `here`), or zero for incoming directions
// of a vacuum face; set is false where the ghost copies the edge cell (outgoing
// directions of a vacuum face).
__device__ __forceinline__ double ghost_value(const StepArgs &p, unsigned at, bool here, int side,
                                              int d, int m, bool incoming, bool &set) {
  const int bc = p.bc[d][side];
  set = bc == kFixed || (bc == kVacuum && incoming);
  double v = 0.0;
  if (bc == kFixed) {
    const double *tab = p.gface[d * 2 + side];
    if (tab) {
      if (here) v = tab[(size_t)m * (size_t)(p.ncell / p.n[d]) + at];
    } else {
      v = p.ghost[(size_t)(d * 2 + side) * p.nang + m];
    }
  }
  return v;
}

// The ghosts among a slot's reads r (offsets -1 or 0, +1, and the upwind far
// cell).  Beyond a face every layer has the value of the face cell, which the
// outermost cell of the stencil holds.
__device__ __forceinline__ void ghost_reads(const StepArgs &p, const unsigned (&idx)[4],
                                            unsigned kinds, int d, int m, bool pos,
                                            double &lo, double &up, double &far) {
  bool set;
  const double gl = ghost_value(p, idx[0], kinds & 1u, 0, d, m, pos, set);
  if (set) {
    lo = kinds & 2u ? gl : lo;
    if (pos) far = kinds & 1u ? gl : far;
  }
  const double gu = ghost_value(p, idx[3], kinds & 8u, 1, d, m, !pos, set);
  if (set) {
    up = kinds & 4u ? gu : up;
    if (!pos) far = kinds & 8u ? gu : far;
  }
}

// The face of one angle (see Face64) from the intensities at offsets 0 and +1
// and at the upwind far cell (-1 for mu > 0, +2 for mu < 0): G relative to the
// lower cell and Gp relative to the upper one.
__device__ __forceinline__ void face_value(const Face64 &f, double n0, double n1, double n2,
                                           double h2, bool pos, double I0, double I1, double If,
                                           double invC, double &G, double &Gp) {
  const double V = n0 * f.w0[0] + n1 * f.w0[1] + n2 * f.w0[2];
  const double Vf = n0 * f.wf[0] + n1 * f.wf[1] + n2 * f.wf[2];
  const double cab = f.ca + f.cb;
  double Vx, dx, k, kp, hs;
  if (pos) {
    Vx = n0 * f.wm[0] + n1 * f.wm[1] + n2 * f.wm[2];
    dx = I0 - If;
    k = f.cb;
    kp = cab;
    hs = h2;
  } else {
    Vx = n0 * f.wp[0] + n1 * f.wp[1] + n2 * f.wp[2];
    dx = If - I1;
    k = cab;
    kp = f.cb;
    hs = -h2;
  }
  const double D = fma_(-V, invC, I1 - I0), Dx = fma_(-Vx, invC, dx);
  const double q = vl_half(Dx, D), qv = vl_half(Vf, V);
  const double slopes = fma_(hs * f.ca, q, f.f * qv);
  G = fma_(k, D, fma_(f.r, V, slopes));
  Gp = fma_(-kp, D, fma_(-f.l, V, slopes));
}

// One lane up: lane l receives lane l - 1's value (lane 0 receives 0).
__device__ __forceinline__ double lane_below(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Plan of a block's LDS, the same on the host (launch size) and the device.
// The build area (face data, start table) and the reduction rows share their
// bytes: barriers separate the uses.
constexpr int kMaxStarts = 9;  // lanes without a lower x neighbour, rows of >= 8 cells
constexpr int kCellRows = 5;   // sigma_a, sigma_s, u
struct Lds64 {
  size_t face_x, both, starts, red_tot, sol, cell, total;
  int nboth, rows;
};
// Rows of values per reduction round: all where the waves' rows fit 64 KB.
__host__ __device__ constexpr int red_rows64(int G) { return G <= 8 ? kRows : G <= 14 ? 7 : 6; }
__host__ __device__ inline Lds64 lds64(int G, int NS, int ndim, bool xs, bool transport) {
  Lds64 l{};
  size_t o = 0;
  l.face_x = o;
  if (xs) o += face_lds_bytes();
  l.both = o;
  l.nboth = ndim - (xs ? 1 : 0);
  o += (size_t)l.nboth * both_lds_bytes();
  l.starts = o;
  if (xs) o += (size_t)G * NS * kMaxStarts * 8;
  l.rows = red_rows64(G);
  if (!transport) {
    size_t r = (size_t)G * l.rows * 64 * 8;
    l.red_tot = r;
    r += (size_t)l.rows * 64 * 8;
    l.sol = r;
    r += 6 * 64 * 8;
    if (r > o) o = r;
    l.cell = o;
    o += (size_t)kCellRows * 64 * 8;
  }
  l.total = o;
  return l;
}

// Transport of the NS angles m0 .. m0 + NS - 1 for one 64-cell tile into
// dF[], one axis at a time.
template <int NS, int PF, bool PER>
struct Transport64 {
  const StepArgs &p;
  const int lane, m0, NA;
  const unsigned c;      // the lane's cell
  const double invC;

  // the planes and records of the wave's angles, opened once per axis
  struct Set {
    const double *I;
    cptr<double> R;
    long long N;
    int last;  // last slot with an angle of its own
    __device__ __forceinline__ cptr<double> rec(int k) const { return R + (unsigned)k * kRec; }
    __device__ __forceinline__ unsigned flags(int k) const {
      return ((cptr<unsigned>)(R + (unsigned)k * kRec + rec_flags))[0];
    }
    // slots past the set read the last plane (their records are zero)
    __device__ __forceinline__ const double *plane(int k) const {
      return I + (k < last ? k : last) * N;
    }
  };
  // The scalars of a slot along axis d, loaded one slot ahead of their use.
  struct Rec {
    double n0, n1, n2, mud, h;
    unsigned fl;
  };
  __device__ static __forceinline__ Rec load_rec(const Set &s, int k, int d) {
    const cptr<double> R = s.rec(k);
    return Rec{R[rec_n0], R[rec_n1], R[rec_n2], R[rec_n0 + d], R[rec_h0 + d], s.flags(k)};
  }
  __device__ __forceinline__ Set open() const {
    const int m = m0 + opaque_zero();
    return Set{static_cast<const double *>(p.I_in) + (long long)m * p.ncell,
               (cptr<double>)(p.arec + (long long)m * kRec), (long long)p.ncell, NA - 1 - m0};
  }

  // One shared axis: every lane forms its high face; below(k, Gp) gives the
  // face below relative to the cell and may keep Gp.
  template <typename Below>
  __device__ __forceinline__ void shared_axis(const Face64 &f, int d,
                                              double (&dF)[NS], Below below) const {
    const Set set = open();
    // some lane of the wave has a ghost cell along this axis (wave-uniform)
    const bool gh = !PER && __any(f.kinds != 0);
    double rq[PF][3];
    auto reads = [&](int k, double (&r)[3]) {
      const double *I = set.plane(k);
      const bool pos = (set.flags(k) >> d) & 1u;
      r[0] = plane_buf_ld(I, f.idx[1]);
      r[1] = plane_buf_ld(I, f.idx[2]);
      r[2] = plane_buf_ld(I, pos ? f.idx[0] : f.idx[3]);
    };
#pragma unroll
    for (int j = 0; j < PF; ++j)
      if (j < NS) reads(j, rq[j]);
    Rec next = load_rec(set, 0, d);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      __builtin_amdgcn_sched_barrier(0);  // keeps the reads ahead where they are
      double r[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) r[t] = rq[k % PF][t];
      if (k + PF < NS) reads(k + PF, rq[k % PF]);
      const Rec R = next;
      if (k + 1 < NS) next = load_rec(set, k + 1, d);
      if (!((R.fl >> (3 + d)) & 1u)) continue;  // mu_d = 0, padding slots
      const bool pos = (R.fl >> d) & 1u;
      const double mud = R.mud;
      if (!PER && gh) ghost_reads(p, f.idx, f.kinds, d, m0 + k, pos, r[0], r[1], r[2]);
      double G, Gp;
      face_value(f, R.n0, R.n1, R.n2, R.h, pos, r[0], r[1], r[2], invC, G, Gp);
      const double lo = below(k, Gp);
      dF[k] = fma_(-mud, G - lo, dF[k]);
    }
  }

  // An axis on which every cell forms both its faces.
  __device__ __forceinline__ void both_axis(const Both64 &s, int d, double (&dF)[NS]) const {
    const Set set = open();
    const bool gh = !PER && __any(s.kinds != 0);
    double rq[PF][4];
    auto reads = [&](int k, double (&r)[4]) {
      const double *I = set.plane(k);
      const bool pos = (set.flags(k) >> d) & 1u;
      r[0] = plane_buf_ld(I, s.idx[1]);
      r[1] = plane_buf_ld(I, s.idx[2]);
      r[2] = plane_buf_ld(I, pos ? s.idx[0] : s.idx[3]);
      r[3] = plane_buf_ld(I, c);
    };
#pragma unroll
    for (int j = 0; j < PF; ++j)
      if (j < NS) reads(j, rq[j]);
    Rec next = load_rec(set, 0, d);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      __builtin_amdgcn_sched_barrier(0);  // keeps the reads ahead where they are
      double r[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) r[t] = rq[k % PF][t];
      if (k + PF < NS) reads(k + PF, rq[k % PF]);
      const Rec R = next;
      if (k + 1 < NS) next = load_rec(set, k + 1, d);
      if (!((R.fl >> (3 + d)) & 1u)) continue;
      const bool pos = (R.fl >> d) & 1u;
      const double n0 = R.n0, n1 = R.n1, n2 = R.n2, mud = R.mud, h2 = R.h;
      if (!PER && gh) ghost_reads(p, s.idx, s.kinds, d, m0 + k, pos, r[0], r[1], r[2]);
      double V[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) V[j] = n0 * s.w[j][0] + n1 * s.w[j][1] + n2 * s.w[j][2];
      const double D1 = fma_(-V[1], invC, r[3] - r[0]);
      const double D2 = fma_(-V[2], invC, r[1] - r[3]);
      const double q0 = vl_half(D1, D2);
      double T;
      if (pos) {
        const double D0 = fma_(-V[0], invC, r[0] - r[2]);
        const double qm = vl_half(D0, D1);
        T = s.cbR * D2 + (s.caL + s.cbL) * D1 + h2 * (s.caR * q0 - s.caL * qm);
      } else {
        const double D3 = fma_(-V[3], invC, r[2] - r[1]);
        const double qp = vl_half(D2, D3);
        T = (s.caR + s.cbR) * D2 + s.cbL * D1 - h2 * (s.caR * qp - s.caL * q0);
      }
      const double qvL = vl_half(s.fL > 0.0 ? V[0] : V[2], V[1]);
      const double qvR = vl_half(s.fR > 0.0 ? V[1] : V[3], V[2]);
      T += s.rR * V[2] + s.lL * V[1] + (s.fR * qvR - s.fL * qvL);
      dF[k] -= mud * T;
    }
  }
};

// The low x faces (relative to the cell) of the lanes that start a run along
// x: lane j nx - x0 for j >= 1 and lane 0, nst of them, for the NS slots of the
// wave, one lane per (slot, start).  tab[k kMaxStarts + j].
template <int NS, bool PER>
__device__ __forceinline__ void start_faces(const StepArgs &p, int cfirst, int climit, int x0,
                                            int nst, int m0, int lane, double *tab) {
  const int nx = p.n[0];
  const double invC = p.invC;
  const unsigned inv = 65536u / (unsigned)nst + 1u;
  for (int b = 0; b < NS * nst; b += 64) {
    const int pr = b + lane;
    const bool on = pr < NS * nst;
    const int k = on ? (int)(((unsigned)pr * inv) >> 16) : 0;
    const int j = on ? pr - k * nst : 0;
    const int m = m0 + k < p.nang ? m0 + k : p.nang - 1;
    // a start past the last cell (no active lane has it) takes the first one
    const int jj = cfirst + j * nx - x0 < climit ? j : 0;
    const int x = jj ? 0 : x0;
    Face64 f;
    load_face64<PER>(p, cfirst - x0 + jj * nx, x - 1, 0, f);
    const double *R = p.arec + (size_t)m * kRec;
    const double mud = R[rec_n0];
    const bool pos = mud > 0.0;
    const double *I = static_cast<const double *>(p.I_in) + (size_t)m * (size_t)p.ncell;
    double r0 = I[f.idx[1]], r1 = I[f.idx[2]], rf = I[pos ? f.idx[0] : f.idx[3]];
    if (!PER && __any(f.kinds != 0)) ghost_reads(p, f.idx, f.kinds, 0, m, pos, r0, r1, rf);
    double G, Gp;
    face_value(f, mud, R[rec_n1], R[rec_n2], R[rec_h0], pos, r0, r1, rf, invC, G, Gp);
    if (on) tab[k * kMaxStarts + j] = Gp;
  }
}

// The 64 cells of a block and what its waves share about them.
template <int NS, bool PER>
struct Tile64 {
  // slots whose plane reads are in flight, as the registers allow
  static constexpr int PF0 = NS <= 8 ? 4 : NS <= 10 ? 3 : 5;
  static constexpr int PF = PF0 < NS ? PF0 : NS;
  using Transport = Transport64<NS, PF, PER>;
  const StepArgs &p;
  const Geo64 &q;
  const Lds64 L;
  char *lds;
  int g, G, lane;
  bool xs, act, start;
  int c;       // the lane's cell; idle lanes shadow the last one
  int first;   // cell of lane 0
  int row, x, x0, nst, mystart;

  __device__ __forceinline__ Tile64(const StepArgs &p_, const Geo64 &q_, int blk, int G_,
                                    char *lds_, bool fused, bool transport)
      : p(p_),
        q(q_),
        L(lds64(G_, NS, p_.ndim, NS >= kSharedSlots && q_.xs && fused, transport)),
        lds(lds_) {
    lane = threadIdx.x & 63;
    // wave-uniform: the wave's angles and their records are scalars
    g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    G = G_;
    xs = NS >= kSharedSlots && q.xs && fused;
    first = blk * 64;
    act = first + lane < p.ncell;
    c = act ? first + lane : p.ncell - 1;
    const int nx = p.n[0];
    row = div_by(c, p.inv_n0);
    x = c - row * nx;
    const int row0 = __builtin_amdgcn_readfirstlane(row);
    x0 = first - row0 * nx;
    nst = 1 + __builtin_amdgcn_readfirstlane(div_by(x0 + 63, p.inv_n0));  // lanes without a
                                                                          // neighbour below
    mystart = row - row0;  // the start of the lane's run
    start = lane == 0 || x == 0;
  }

  // Face data of the tile into LDS, one axis a wave; with_cell: also the
  // cell's opacities and velocity estimate (Step 3).
  __device__ __forceinline__ void build(bool with_axes, bool with_cell) const {
    const int nax = with_axes ? p.ndim : 0;
    for (int d = g; d < nax + (with_cell ? 1 : 0); d += G) {
      // the cell index made anew in every turn: addresses formed from it are
      // not worth registers over the loop
      int cc = c;
      asm volatile("" : "+v"(cc));
      if (d == nax) {
        cell(cc);
      } else if (xs && d == 0) {
        Face64 f;
        load_face64<PER>(p, cc - x, x, 0, f);
        face_put(lds + L.face_x, f, lane);
      } else {
        const int z = div_by(row, p.inv_n1);
        const int k = d == 0 ? x : d == 1 ? row - z * p.n[1] : z;
        Both64 b;
        load_both64<PER>(p, cc, k, d, b);
        both_put(lds + L.both + (size_t)(d - (xs ? 1 : 0)) * both_lds_bytes(), b, lane);
      }
    }
  }

  __device__ __forceinline__ void cell(int c) const {
    const size_t N = (size_t)p.ncell;
    const double dt = p.dt, C = p.C, P = p.P;
    const double sa = p.sa[c], ss = p.ss[c], rho = p.rho[c];
    double u0 = p.v[c], u1 = p.v[N + c], u2 = p.v[2 * N + c];
    if (p.estimate_v) {
      const double h = 0.5 * dt * (sa + ss);
      const double E = p.mom_in[c];
      const double F0 = p.mom_in[N + c], F1 = p.mom_in[2 * N + c], F2 = p.mom_in[3 * N + c];
      const double P0 = p.mom_in[4 * N + c], P1 = p.mom_in[5 * N + c], P2 = p.mom_in[6 * N + c];
      const double base = rho + h * C * rho, hPC = h * P * p.invC;
      u0 = (rho * u0 + h * (C * rho * u0 + P * F0)) * fast_rcp(base + hPC * (E + P0));
      u1 = (rho * u1 + h * (C * rho * u1 + P * F1)) * fast_rcp(base + hPC * (E + P1));
      u2 = (rho * u2 + h * (C * rho * u2 + P * F2)) * fast_rcp(base + hPC * (E + P2));
    }
    double *s = reinterpret_cast<double *>(lds + L.cell) + lane;
    s[0] = sa;
    s[64] = ss;
    s[128] = u0;
    s[192] = u1;
    s[256] = u2;
  }

  __device__ __forceinline__ double *table() const {
    return reinterpret_cast<double *>(lds + L.starts) + (size_t)g * NS * kMaxStarts;
  }
  __device__ __forceinline__ void starts(int m0) const {
    start_faces<NS, PER>(p, first, p.ncell, x0, nst, m0, lane, table());
  }

  // Increments of the angles m0 .. into dF (zero on entry).
  __device__ __forceinline__ void transport(int m0, double (&dF)[NS]) const {
    const Transport tr{p, lane, m0, p.nang, (unsigned)c, p.invC};
    if (xs) {
      Face64 f;
      face_get(lds + L.face_x, p.dt_dx[0], f, lane);
      const double *tab = table() + mystart;
      tr.shared_axis(f, 0, dF, [&](int k, double Gp) {
        const double s = tab[k * kMaxStarts], b = lane_below(Gp);
        return start ? s : b;
      });
    }
    for (int d = xs ? 1 : 0; d < p.ndim; ++d) {
      Both64 b;
      both_get(lds + L.both + (size_t)(d - (xs ? 1 : 0)) * both_lds_bytes(), b, lane);
      tr.both_axis(b, d, dF);
    }
  }
};

template <int NS, bool PER, int MODE, bool SO, bool STAGED>
struct Step64 {
  using Tile = Tile64<NS, PER>;
  static_assert(!STAGED || NS < kSharedSlots, "the table of low x faces holds one chunk");

  // The transport increment alone.
  __device__ static __forceinline__ void transport(const StepArgs &p, const Geo64 &q, int blk,
                                                   int chunk, int G, char *lds) {
    const Tile t(p, q, blk, G, lds, true, true);
    double *dF = static_cast<double *>(p.dF_out);
    const int m0 = __builtin_amdgcn_readfirstlane((chunk * G + t.g) * NS);
    double pk[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) pk[k] = 0.0;
    t.build(true, false);
    if (t.xs) t.starts(m0);
    __syncthreads();
    t.transport(m0, pk);
    if (t.act) {
#pragma unroll
      for (int k = 0; k < NS; ++k)
        if (m0 + k < p.nang)
          stream_store(&dF[(size_t)(m0 + k) * (size_t)p.ncell + t.c], pk[k]);
    }
  }

  __device__ static __forceinline__ void run(const StepArgs &p, const Geo64 &q, int blk, int G,
                                             char *lds) {
    const Tile t(p, q, blk, G, lds, MODE == kFused64, false);
    const Lds64 &L = t.L;
    double *sbuf = reinterpret_cast<double *>(lds);
    double *stot = reinterpret_cast<double *>(lds + L.red_tot);
    double *ssol = reinterpret_cast<double *>(lds + L.sol);
    double *scell = reinterpret_cast<double *>(lds + L.cell);
    const int lane = t.lane, g = t.g, NA = p.nang, c = t.c;
    // the output fields and totals of this wave: those with number g mod G
    unsigned mine = 0u;
    for (int f = g; f < 28; f += G) mine |= 1u << f;
    const bool act = t.act;
    const size_t N = (size_t)p.ncell;
    const double *Iin = static_cast<const double *>(p.I_in);
    double *Iout = static_cast<double *>(p.I_out);
    const double C = p.C, P = p.P, dt = p.dt, iC = p.invC;
    double pk[NS];  // transport increments, then p_m
    double fs[SO ? 1 : 13];
    double sm[SO ? kNsum : 1];
    if constexpr (SO) {
#pragma unroll
      for (int r = 0; r < kNsum; ++r) sm[r] = 0.0;
    } else {
#pragma unroll
      for (int r = 0; r < 13; ++r) fs[r] = 0.0;
    }
    double u0, u1, u2, sa, ss;
    const int nch = STAGED ? q.chunks : 1;
    double Sa[kChunk], Sb[kChunk], fold[SO ? 1 : 13];
    double ua0, ua1, ua2, uua;
    int it_first = 0;
    bool conv_first = true;
    double rho = 0.0, Tn = 0.0, v0 = 0.0, v1 = 0.0, v2 = 0.0;

    for (int ch = 0; ch < nch; ++ch) {
      const int m0 = STAGED ? (ch * G + g) * NS : g * NS;
#pragma unroll
      for (int k = 0; k < NS; ++k) pk[k] = 0.0;
      if (ch == 0) t.build(MODE == kFused64, true);
      if (MODE == kFused64 && t.xs) t.starts(m0);
      if (ch == 0) __syncthreads();
      // -------------------------------------------- phase A: transport
      if constexpr (MODE == kFused64) {
        t.transport(m0, pk);
      } else {
        const double *dFin = static_cast<const double *>(p.dF_in);
        if (dFin) {
#pragma unroll
          for (int k = 0; k < NS; ++k)
            if (m0 + k < NA) pk[k] = dFin[(size_t)(m0 + k) * N + c];
        }
      }
      const int mo0 = m0 + opaque_zero();
      const cptr<double> Rg = (cptr<double>)(p.arec + (size_t)mo0 * kRec);
      const double *Ig = Iin + (size_t)mo0 * N;

      // -------------------------------------- phase B: source sums
      sa = scell[lane];
      ss = scell[64 + lane];
      u0 = scell[128 + lane];
      u1 = scell[192 + lane];
      u2 = scell[256 + lane];
      const double dsa = dt * sa, dss = dt * ss;
      const double D0 = 1.0 + dsa * C, AW0 = 1.0 + dss * C;
      const bool to5 = ss > sa;  // Step 2 routing: r = I + g4 dF, p = r/D + g5 dF
      const double g4 = to5 ? 0.0 : 1.0, g5 = to5 ? 1.0 : 0.0;
      if constexpr (!SO) {
        constexpr int PB = NS < 4 ? NS : 4;
        double rq[PB];
        const int last = NA - 1 - m0;
        auto own = [&](int k) {
          return plane_buf_ld(Ig + (long long)(k < last ? k : last) * (long long)N, (unsigned)c);
        };
#pragma unroll
        for (int k = 0; k < PB; ++k) rq[k] = own(k);
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const double I = rq[k % PB];
          if (k + PB < NS) rq[k % PB] = own(k + PB);
          if (m0 + k >= NA) continue;
          const cptr<double> R = Rg + (unsigned)k * kRec;
          const double t = R[rec_n0] * u0 + R[rec_n1] * u1 + R[rec_n2] * u2;
          const double D = fma_(-dsa, t, D0), aw = fma_(-dss, t, AW0);
          const double rDa = fast_rcp(D * aw);
          const double invD = aw * rDa, invaw = D * rDa;
          const double r4 = fma_(g4, pk[k], I), d5 = g5 * pk[k];
          const double pm = fma_(r4, invD, d5);
          if constexpr (STAGED) {
            if (act) Iout[(size_t)(m0 + k) * N + c] = pm;
          } else
            pk[k] = pm;
          const double wt2 = R[rec_w] * t * t;
          const double xx = wt2 * invD, y = wt2 * invaw, zz = y * t;
          fs[0] = fma_(R[rec_w], r4, fs[0]);
          fs[1] = fma_(R[rec_wn0], r4, fs[1]);
          fs[2] = fma_(R[rec_wn1], r4, fs[2]);
          fs[3] = fma_(R[rec_wn2], r4, fs[3]);
          fs[4] = fma_(R[rec_w], d5, fs[4]);
          fs[5] = fma_(R[rec_wn0], d5, fs[5]);
          fs[6] = fma_(R[rec_wn1], d5, fs[6]);
          fs[7] = fma_(R[rec_wn2], d5, fs[7]);
          fs[8] = fma_(xx, r4, fs[8]);
          fs[9] = fma_(y, pm, fs[9]);
          fs[10] = fma_(xx, t, fs[10]);
          fs[11] += zz;
          fs[12] = fma_(zz, invD, fs[12]);
        }
      }
    }
    const double uu = u0 * u0 + u1 * u1 + u2 * u2;
    const double dsa = dt * sa, dss = dt * ss;
    const double D0 = 1.0 + dsa * C, E0 = dsa * C, AW0 = 1.0 + dss * C;
    const double B0 = -dss * C - dss * uu * iC, dssC = dss * iC;
    const double kap = dsa * iC;
    ua0 = u0, ua1 = u1, ua2 = u2, uua = uu;
    if (g == 0 || SO) {
      rho = p.rho[c];
      Tn = p.T[c];
    }
    const double cv = rho * p.cvfac;
    const int m0 = g * NS;
    const cptr<double> Rg = (cptr<double>)(p.arec + (size_t)(m0 + opaque_zero()) * kRec);
    const double *Ig = Iin + (size_t)m0 * N;
    __syncthreads();  // the reductions reuse the bytes of the build area
    if constexpr (SO) {
      so_sums(p, G, g, lane, NA, m0, c, Rg, Ig, pk, sm, sbuf, stot, u0, u1, u2, uu, dsa, dss, D0,
              E0, AW0, B0, dssC, kap, cv, rho, Tn, sa, ss, ua0, ua1, ua2, uua, it_first,
              conv_first, Sa, Sb);
    } else {
#pragma unroll
      for (int r = 0; r < 13; ++r) fold[r] = fs[r];
      reduce<13, false>(fold, sbuf, stot, g, G, lane);
      Sb[8] = fold[1] + fold[5];
      Sb[9] = fold[2] + fold[6];
      Sb[10] = fold[3] + fold[7];
    }

    // --------------------------------------------- solve (wave 0)
    double X = 0.0, kQ = 0.0, s1 = 0.0, s2 = 0.0, T = 0.0, newton_it = 0.0;
    if (g == 0) {
      if constexpr (!SO)
        unfold_sums(fold, p.wmom, u0, u1, u2, uu, D0, dsa, E0, AW0, dss, B0, dssC, Sa, Sb);
      double Q;
      int it;
      bool conv;
      T = absorb_solve(p, Sa, kap, uua, cv, Tn, sa, X, Q, it, conv);
      if (SO) {
        it = it > it_first ? it : it_first;
        conv = conv && conv_first;
      }
      if (act && (!conv || !(T > 0.0) || !isfinite(T))) atomicOr(p.status, 1);
      kQ = kap * Q;
      const double Sbr = Sa[9] + X * Sb[4] - kQ * Sb[5];
      const double Sr5 = Sa[10] + X * Sb[6] - kQ * Sb[7];
      const double a11 = 1.0 + Sb[0], a12 = Sb[1], a21 = Sb[2], a22 = 1.0 + Sb[3];
      const double idet = fast_rcp(a11 * a22 - a12 * a21);
      s1 = (Sbr * a22 - a12 * Sr5) * idet;
      s2 = (a11 * Sr5 - a21 * Sbr) * idet;
      newton_it = double(it);
      ssol[0 * 64 + lane] = X;
      ssol[1 * 64 + lane] = kQ;
      ssol[2 * 64 + lane] = s1;
      ssol[3 * 64 + lane] = s2;
      ssol[4 * 64 + lane] = T;
      ssol[5 * 64 + lane] = newton_it;
    }
    __syncthreads();
    X = ssol[lane];
    kQ = ssol[64 + lane];
    s1 = ssol[128 + lane];
    s2 = ssol[192 + lane];
    T = ssol[256 + lane];
    newton_it = ssol[320 + lane];

    // fields of the outputs, loaded here so that their latency overlaps
    // phase C
    rho = p.rho[c];
    Tn = p.T[c];
    v0 = p.v[c];
    v1 = p.v[N + c];
    v2 = p.v[2 * N + c];
    double accE = 0.0, accM[3] = {0.0, 0.0, 0.0};
    if (p.accumulate) {
      if (p.dEgas && (mine >> 14) & 1u) accE = p.dEgas[c];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (p.dMom && (mine >> (15 + k)) & 1u) accM[k] = p.dMom[(size_t)k * N + c];
    }

    // --------------------------------------- phase C: new intensities
    double mo[kChunk];
#pragma unroll
    for (int r = 0; r < 10; ++r) mo[r] = 0.0;
    mo[10] = 1.0e300;
    for (int ch = 0; ch < nch; ++ch) {
      const int mc = STAGED ? (ch * G + g) * NS : m0;
      const cptr<double> Rc = STAGED ? (cptr<double>)(p.arec + (size_t)mc * kRec) : Rg;
      double *Og = Iout + (size_t)mc * N;
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (mc + k >= NA) continue;
        const cptr<double> R = Rc + (unsigned)k * kRec;
        const double t = R[rec_n0] * u0 + R[rec_n1] * u1 + R[rec_n2] * u2;
        const double ta = SO ? R[rec_n0] * ua0 + R[rec_n1] * ua1 + R[rec_n2] * ua2 : t;
        const double D = fma_(-dsa, ta, D0), aw = fma_(-dss, t, AW0);
        const double rDa = fast_rcp(D * aw);
        const double e = fma_(3.0 * dsa, ta, E0), cm = -3.0 * dss * t;
        const double pm = STAGED ? Og[(size_t)(unsigned)k * N + c] : pk[k];
        // I' = invaw (p - s1 - c s2) + invD invaw (e X - kappa Q)
        const double In = D * rDa * (pm - s1 - cm * s2) + rDa * (e * X - kQ);
        if (act) stream_store(&Og[(size_t)(unsigned)k * N + c], In);
#pragma unroll
        for (int r = 0; r < 10; ++r) mo[r] = fma_(R[rec_w + r], In, mo[r]);
        mo[10] = In < mo[10] ? In : mo[10];
      }
    }
    reduce<kChunk, true>(mo, sbuf, stot, g, G, lane);
#pragma unroll
    for (int r = 0; r < 10; ++r) mo[r] *= kFourPi;

    // ------------------------------------------------ Step 7 and outputs
    const double PC = P * iC, f4 = kFourPi * PC, gf = p.gasfac;
    const double irho = fast_rcp(rho);
    const double dm0 = gf * (-PC * mo[1] + f4 * Sb[8]);
    const double dm1 = gf * (-PC * mo[2] + f4 * Sb[9]);
    const double dm2 = gf * (-PC * mo[3] + f4 * Sb[10]);
    const double mm0 = rho * v0, mm1 = rho * v1, mm2 = rho * v2;
    const double ek = (((mm0 + dm0) * (mm0 + dm0) + (mm1 + dm1) * (mm1 + dm1) +
                        (mm2 + dm2) * (mm2 + dm2)) -
                       (mm0 * mm0 + mm1 * mm1 + mm2 * mm2)) *
                      (0.5 * irho);
    const double cvg = rho * p.cvfac * gf;
    const double deg = cvg * (T - Tn) + ek;
    const double vn0 = p.feedback ? v0 + dm0 * irho : v0;
    const double vn1 = p.feedback ? v1 + dm1 * irho : v1;
    const double vn2 = p.feedback ? v2 + dm2 * irho : v2;
    if (act) {
      // field f (0-9 the moments, 10-12 3vJ of the new state, 13 T, 14
      // dEgas, 15-17 dMom, 18-27 the output moments) by wave f mod G
#pragma unroll
      for (int f = 0; f < 28; ++f) {
        if (!((mine >> f) & 1u)) continue;
        double val;
        double *dst;
        if (f < 10) {
          val = mo[f];
          dst = p.mom_out + (size_t)f * N;
        } else if (f < 13) {
          val = p.ivfac * (f == 10 ? vn0 : f == 11 ? vn1 : vn2) * mo[0] * (1.0 / kFourPi);
          dst = p.mom_out + (size_t)f * N;
        } else if (f == 13) {
          val = T;
          dst = p.T;
        } else if (f == 14) {
          if (!p.dEgas) continue;
          val = accE + deg;
          dst = p.dEgas;
        } else if (f < 18) {
          if (!p.dMom) continue;
          const int k = f - 15;
          val = accM[k] + (k == 0 ? dm0 : k == 1 ? dm1 : dm2);
          dst = p.dMom + (size_t)k * N;
        } else if (f == 18) {
          if (!p.oE) continue;
          val = mo[0];
          dst = p.oE;
        } else if (f < 22) {
          if (!p.oF) continue;
          val = mo[f - 18];
          dst = p.oF + (size_t)(f - 19) * N;
        } else {
          if (!p.oP) continue;
          val = mo[f - 18];
          dst = p.oP + (size_t)(f - 22) * N;
        }
        stream_store(&dst[c], val);
      }
      // gas feedback: the new velocity (every wave has read this cell's v
      // before the reductions above; the next step's tables are built from it)
      if (p.feedback && g == G - 1) {
        p.v[c] = vn0;
        p.v[N + c] = vn1;
        p.v[2 * N + c] = vn2;
      }
    }
    // the tile's totals, component k by wave k mod G (on one wave they are
    // a tail of 12 shuffle trees in which the other waves idle)
#pragma unroll
    for (int k = 0; k < kNtot; ++k) {
      if (!((mine >> k) & 1u)) continue;
      double s = k == 0   ? P * mo[0]
                 : k == 1 ? cvg * T
                 : k == 2 ? deg
                 : k == 3 ? ek
                 : k < 7  ? (k == 4 ? dm0 : k == 5 ? dm1 : dm2)
                 : k < 10 ? PC * mo[k - 6]
                 : k == 10 ? mo[10]
                           : newton_it;
      if (k < 10) s *= p.vol;
      if (!act) s = tot_init(k);
      s = tot_lanes(k, s);
      if (lane == 0) store_partial(p.partials, p.nparts, blk, k, s, p.accumulate);
    }
  }

  template <int NV, bool MINLAST>
  __device__ static __forceinline__ void reduce(double (&x)[NV], double *buf, double *tot, int g,
                                                int G, int lane) {
    if (G == 1) return;
    if (G <= 8)
      waves_reduce<NV, MINLAST, kRows>(x, buf, tot, g, G, lane);
    else if (G <= 14)
      waves_reduce<NV, MINLAST, 7>(x, buf, tot, g, G, lane);
    else
      waves_reduce<NV, MINLAST, 6>(x, buf, tot, g, G, lane);
  }

  // Second order: the first solve at u gives the time-centred velocity, then
  // the 22 sums with the absorption coefficients at it and the scattering ones
  // at u.
  __device__ static __forceinline__ void so_sums(
      const StepArgs &p, int G, int g, int lane, int NA, int m0, int c, cptr<double> Rg,
      const double *Ig, double (&pk)[NS], double (&sm)[SO ? kNsum : 1], double *sbuf, double *stot,
      double u0, double u1, double u2, double uu, double dsa, double dss, double D0, double E0,
      double AW0, double B0, double dssC, double kap, double cv, double rho, double Tn, double sa,
      double ss, double &ua0, double &ua1, double &ua2, double &uua, int &it_first,
      bool &conv_first, double (&Sa)[kChunk], double (&Sb)[kChunk]) {
    if constexpr (SO) {
      const size_t N = (size_t)p.ncell;
      const double C = p.C;
      const bool to5 = ss > sa;
      const double g4 = to5 ? 0.0 : 1.0, g5 = to5 ? 1.0 : 0.0;
      double s1a[9], hm[9];
#pragma unroll
      for (int r = 0; r < 9; ++r) s1a[r] = hm[r] = 0.0;
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (m0 + k >= NA) continue;
        const cptr<double> R = Rg + (unsigned)k * kRec;
        const double n0 = R[rec_n0], n1 = R[rec_n1], n2 = R[rec_n2];
        const double t = n0 * u0 + n1 * u1 + n2 * u2;
        const double invD = fast_rcp(D0 - dsa * t);
        const double e = E0 + 3.0 * dsa * t;
        const double gg = uu + t * t;
        const double r4 = plane_buf_ld(Ig + (size_t)(unsigned)k * N, (unsigned)c) + g4 * pk[k];
        const double WD = R[rec_w] * invD;
        s1a[0] += WD * r4;
        s1a[1] += WD * e;
        s1a[2] += WD;
        s1a[3] += WD * t * r4;
        s1a[4] += WD * t * e;
        s1a[5] += WD * t;
        s1a[6] += WD * gg * r4;
        s1a[7] += WD * gg * e;
        s1a[8] += WD * gg;
        const double wr = -(WD * dsa * (C - t) * r4), we = WD * e;
        const double nn[3] = {n0, n1, n2};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          hm[j] += nn[j] * wr;
          hm[3 + j] += nn[j] * we;
          hm[6 + j] += nn[j] * WD;
        }
      }
      reduce<9, false>(s1a, sbuf, stot, g, G, lane);
      reduce<9, false>(hm, sbuf, stot, g, G, lane);
      double X1, Q1;
      absorb_solve(p, s1a, kap, uu, cv, Tn, sa, X1, Q1, it_first, conv_first);
      // the Step 4 momentum change of the first solution, as the gas sees it
      const double fm = -p.gasfac * kFourPi * p.P * p.invC, h2r = 0.5 * fast_rcp(rho);
      const double v0 = p.v[c], v1 = p.v[N + c], v2 = p.v[2 * N + c];
      ua0 = v0 + fm * (hm[0] + X1 * hm[3] - kap * Q1 * hm[6]) * h2r;
      ua1 = v1 + fm * (hm[1] + X1 * hm[4] - kap * Q1 * hm[7]) * h2r;
      ua2 = v2 + fm * (hm[2] + X1 * hm[5] - kap * Q1 * hm[8]) * h2r;
      uua = ua0 * ua0 + ua1 * ua1 + ua2 * ua2;
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (m0 + k >= NA) continue;
        const cptr<double> R = Rg + (unsigned)k * kRec;
        const double n0 = R[rec_n0], n1 = R[rec_n1], n2 = R[rec_n2];
        const double Wm = R[rec_w];
        const double t = n0 * u0 + n1 * u1 + n2 * u2;      // scattering
        const double ta = n0 * ua0 + n1 * ua1 + n2 * ua2;  // absorption
        const double D = D0 - dsa * ta, aw = AW0 - dss * t;
        const double rDa = fast_rcp(D * aw);
        const double invD = aw * rDa, invaw = D * rDa;
        const double e = E0 + 3.0 * dsa * ta;
        const double gg = uua + ta * ta;
        const double b = B0 + 2.0 * dss * t - dssC * t * t;
        const double cm = -3.0 * dss * t;
        const double dF = pk[k];
        const double I = plane_buf_ld(Ig + (size_t)(unsigned)k * N, (unsigned)c);
        const double r4 = I + g4 * dF;
        const double pm = r4 * invD + g5 * dF;
        pk[k] = pm;
        const double WD = Wm * invD, Wa = Wm * invaw, Wad = Wa * invD;
        sm[0] += WD * r4;
        sm[1] += WD * e;
        sm[2] += WD;
        sm[3] += WD * ta * r4;
        sm[4] += WD * ta * e;
        sm[5] += WD * ta;
        sm[6] += WD * gg * r4;
        sm[7] += WD * gg * e;
        sm[8] += WD * gg;
        sm[9] += Wa * b * pm;
        sm[10] += Wa * pm;
        sm[11] += Wa * b;
        sm[12] += Wa * b * cm;
        sm[13] += Wa;
        sm[14] += Wa * cm;
        sm[15] += Wad * b * e;
        sm[16] += Wad * b;
        sm[17] += Wad * e;
        sm[18] += Wad;
        const double Ir = I + dF;
        sm[19] += R[rec_wn0] * Ir;
        sm[20] += R[rec_wn1] * Ir;
        sm[21] += R[rec_wn2] * Ir;
      }
#pragma unroll
      for (int r = 0; r < kChunk; ++r) {
        Sa[r] = sm[r];
        Sb[r] = sm[kChunk + r];
      }
      reduce<kChunk, false>(Sa, sbuf, stot, g, G, lane);
      reduce<kChunk, false>(Sb, sbuf, stot, g, G, lane);
    }
  }
};

// Instances: up to ten slots per wave fit 128 registers (four waves per
// SIMD, blocks of up to 16 waves), more take 168 (three, 12 waves).
template <int NS, bool PER, int MODE, bool SO, bool STAGED>
__global__ __launch_bounds__(64 * max_waves64(NS), NS <= 10 ? 4 : 3) void k_step64(StepArgs p,
                                                                                  Geo64 q) {
  extern __shared__ double lds_[];
  const int blk = slab_block((int)blockIdx.x, (int)gridDim.x, p.n, 4);
  Step64<NS, PER, MODE, SO, STAGED>::run(p, q, blk, blockDim.x >> 6,
                                                reinterpret_cast<char *>(lds_));
}

// The transport increment alone (rt_transport): the same faces, written to
// dF_out; the angle chunks of a tile are separate blocks (blockIdx.y).  The step's
// arguments, the first of the kernel, are read where the launch put them: from the
// parameter itself, whose tables the ghosts index by axis, the compiler made a copy
// in scratch memory in the non-periodic instances of 20 and more angles (900 B and
// 120 to 280 registers spilled a lane; 96 x 96 x 48 S8 between fixed, vacuum and copy
// faces, transport and source: 1.76 ms so, 0.79 as it is).
template <int NS, bool PER>
__global__ __launch_bounds__(64 * max_waves64(NS), NS <= 10 ? 4 : 3) void k_transport64(StepArgs,
                                                                                       Geo64 q) {
  extern __shared__ double lds_[];
  const StepArgs &p = *(const StepArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  const int blk = slab_block((int)blockIdx.x, (int)gridDim.x, p.n, 4);
  Step64<NS, PER, kFused64, false, false>::transport(p, q, blk, (int)blockIdx.y,
                                                            blockDim.x >> 6,
                                                            reinterpret_cast<char *>(lds_));
}

}  // namespace rtk
