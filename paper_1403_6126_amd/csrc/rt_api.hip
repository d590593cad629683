// Host side of the context API declared in include/rt.h: validation,
// device-memory plan, and the launches of the per-call and per-step kernels.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "rt.h"
#include "rt_cellwise.hpp"
#include "rt_internal.hpp"

namespace rtk {

// Interface table, per-call angle factors and IV basis (once per call).
// faces[(d*3 + j)*ncell + c] for the face between the cell below c along
// axis d (wrapped; the edge cell itself at a non-periodic low boundary,
// whose ghost copies it) and c, with the face opacity and flow speed u the
// means of the two cells (Section 4.2):
//   j = 0  C alpha, the transport speed factor times C;
//   j = 1  the lower cell's share of the centred IV value: 1 when the flow
//          goes up the axis (u > 0, upwind = lower cell), 0 when it goes
//          down, 1/2 at u = 0 (centred);
//   j = 2  the signed van Leer factor of the IV value, sign(u) (1 - nu_v),
//          nu_v = |u| dt/dx (0 at u = 0).
// arec[m*kRec + f] (and FP32 copies unless arecf is null) are the per-angle records of the
// call: direction, 1 - C |mu_d| dt/dx_d, w, w n_d, w n_i n_j and the sign
// bits of the direction (as integers in the slot's low word); records
// nang .. nrec-1 (the padding slots of the wave-group kernel) are zero.
// wv = 3 v E/(4pi) of the current moments into mom[10..12].  One thread per
// cell and per record (max of the two).
__global__ __launch_bounds__(kBlock) void k_faces(StepArgs p, double *faces, double *mom,
                                                  double *arec, float *arecf, int nrec) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c < nrec) {
    double r[kRec];
    for (int f = 0; f < kRec; ++f) r[f] = 0.0;
    if (c < p.nang) {
      const double n[3] = {p.mu[c], p.mu[p.nang + c], p.mu[2 * p.nang + c]};
      const double w = p.w[c];
      for (int d = 0; d < 3; ++d) {
        r[rec_n0 + d] = n[d];
        r[rec_h0 + d] = 1.0 - p.C * fabs(n[d]) * p.dt_dx[d];
        r[rec_wn0 + d] = w * n[d];
      }
      r[rec_w] = w;
      r[rec_wnn + 0] = w * n[0] * n[0];
      r[rec_wnn + 1] = w * n[1] * n[1];
      r[rec_wnn + 2] = w * n[2] * n[2];
      r[rec_wnn + 3] = w * n[0] * n[1];
      r[rec_wnn + 4] = w * n[0] * n[2];
      r[rec_wnn + 5] = w * n[1] * n[2];
    }
    // the signs of the direction as integer bits (the step kernel tests
    // them on the scalar unit, which has no floating-point compare)
    unsigned flags = 0;
    for (int d = 0; d < 3; ++d) {
      if (r[rec_n0 + d] > 0.0) flags |= 1u << d;
      if (r[rec_n0 + d] != 0.0) flags |= 8u << d;
    }
    for (int f = 0; f < kRec; ++f) {
      if (f == rec_flags) {
        unsigned long long bits = flags;
        arec[(size_t)c * kRec + f] = __longlong_as_double((long long)bits);
        if (arecf) arecf[(size_t)c * kRec + f] = __uint_as_float(flags);
      } else {
        arec[(size_t)c * kRec + f] = r[f];
        if (arecf) arecf[(size_t)c * kRec + f] = float(r[f]);
      }
    }
  }
  if (c >= p.ncell) return;
  const size_t N = (size_t)p.ncell;
  const double sig_c = p.sa[c] + p.ss[c];
  const int q[3] = {c % p.n[0], (c / p.n[0]) % p.n[1], c / (p.n[0] * p.n[1])};
  for (int d = 0; d < p.ndim; ++d) {
    int cl;
    if (q[d] > 0)
      cl = c - p.stride[d];
    else if (p.bc[d][0] == kPeriodic)
      cl = c + (p.n[d] - 1) * p.stride[d];
    else
      cl = c;
    const double sig = 0.5 * ((p.sa[cl] + p.ss[cl]) + sig_c);
    const double u = 0.5 * (p.v[(size_t)d * N + cl] + p.v[(size_t)d * N + c]);
    faces[(size_t)(d * 3 + 0) * N + c] = p.C * alpha_of(sig, p.dl10[d]);
    faces[(size_t)(d * 3 + 1) * N + c] = iv_lower_share(u);
    faces[(size_t)(d * 3 + 2) * N + c] = iv_signed_factor(u, p.dt_dx[d]);
  }
  const double J = mom[c] * (1.0 / kFourPi);
  for (int k = 0; k < 3; ++k) mom[(size_t)(10 + k) * N + c] = p.ivfac * p.v[(size_t)k * N + c] * J;
}

// Sets one int in device memory (status words; a kernel, not a memset, so
// that a captured graph replays it correctly).
__global__ void k_set_int(int *p, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// Totals of the partial rows, first stage: block b reduces chunk b of the nb
// rows into out[k*gridDim.x + b], wave k component k.  With one chunk that is
// the result; otherwise k_totals_join reduces the chunk rows.  One workgroup
// that read every row took 165 us on the 32768 rows of the 128^3 box (a chain
// of loads on one CU) and 1.3 ms on those of the 256^3 box; a block per chunk
// reads them on all CUs.
__global__ __launch_bounds__(64 * kNtot) void k_totals(const double *partials, int nb,
                                                       double *out) {
  const int lane = threadIdx.x & 63, k = threadIdx.x >> 6, c = blockIdx.x;
  const int r0 = c * kTotChunk, r1 = r0 + kTotChunk < nb ? r0 + kTotChunk : nb;
  const double s = tot_rows(partials + (size_t)k * nb, r0, r1, k, lane);
  if (lane == 0) out[(size_t)k * gridDim.x + c] = s;
}

// Second stage: the chunk rows [kNtot][nch], lane c % 64 taking chunk c.
__global__ __launch_bounds__(64 * kNtot) void k_totals_join(const double *chunks, int nch,
                                                            double *out) {
  const int lane = threadIdx.x & 63, k = threadIdx.x >> 6;
  double s = tot_init(k);
  for (int c = lane; c < nch; c += 64) s = tot_op(k, s, chunks[(size_t)k * nch + c]);
  s = tot_lanes(k, s);
  if (lane == 0) out[k] = s;
}

// I[m][c] = T[c]^4 / (4 pi), the equilibrium intensity in every direction.
template <typename S>
__global__ __launch_bounds__(kBlock) void k_equilibrium(const double *T, S *I, int ncell,
                                                        int nang) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= ncell) return;
  const double t = T[c];
  const S b = S((t * t) * (t * t) / kFourPi);
  for (int m = 0; m < nang; ++m) I[(size_t)m * ncell + c] = b;
}

namespace {

bool hip_ok(hipError_t e) { return e == hipSuccess; }

// Kernel launches report failure through hipGetLastError only; an error left
// by an earlier call of this thread (already returned by that call) is
// cleared first so that the check after a launch sees only the launch.
void clear_stale_error() { (void)hipGetLastError(); }

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Launch shape with FP32 intensities: the angle groups are dealt to four waves
// (more groups per wave amortise the per-cell work of a wave over more
// angles), and to up to kMaxWaves when the groups would not fit
// kMaxGroupsPerWave per wave; more directions run on the thread-per-cell
// kernel.  The sums of a cell are FP32 chains over a wave's angles, so the
// shape also fixes their order.
void pick_shape32(int nang, KShape &k) {
  const int ng = (nang + kAnglesPerWave - 1) / kAnglesPerWave;
  int G = ng < 4 ? ng : 4;
  int NG = (ng + G - 1) / G;
  if (NG > kMaxGroupsPerWave) {
    G = ng < kMaxWaves ? ng : kMaxWaves;
    NG = (ng + G - 1) / G;
  }
  if (NG <= kMaxGroupsPerWave) {
    k.waves = G;
    k.groups = NG;
  }
}

constexpr int kSlots64[] = {
#define RT_ITEM(ns) ns,
    RT_SLOTS64(RT_ITEM)
#undef RT_ITEM
};

// Smallest number of angles per wave that is built and holds n (0 if none).
int slots64_for(int n) {
  for (int s : kSlots64)
    if (s >= n) return s;
  return 0;
}

// Launch shape with FP64 intensities: waves per block and angles per wave.
//   * One wave for up to 4 directions; else blocks of 4 waves and as many angles per wave
//     as that takes: the work a wave does once per tile is worth about ten
//     angles, and blocks of four fill the four SIMDs evenly, three to a CU.  One
//     step of the 128^3 S8 box takes 2.2 ms with 4 x 20, 2.4 ms with 8 x 10 and
//     3.6 ms and more with 5, 6, 7 or 10 waves, of which a CU then holds one
//     block.  100^3 S2: 4 x 2 0.27 ms, 2 x 4 0.32; 512 x 256 with 90 directions:
//     4 x 24 0.18 ms, 8 x 12 0.26.
//   * More than 120 directions: 12 waves, the most that three waves per SIMD
//     allow (80^3 S12: 12 x 15 1.4 ms, 8 x 24 1.7; S10: 4 x 30 0.88, 12 x 10 1.03,
//     8 x 15 1.08).
//   * Up to 256 tiles (one a CU at most) the time of a step is that of one
//     wave: up to 16 waves, two angles each or more (512 cells, 16 directions,
//     100 steps: 8 x 2 1.18 ms, 16 x 1 1.29, 2 x 8 1.61; 16^3 S8 16 x 5 0.17 ms,
//     4 x 20 0.21).
//   * Sets that do not fit (more than 360 directions) run in chunks of
//     kStagedSlots angles per wave.
// Sharing the faces along x costs a wave one pass of about 13 angles' gain per 64
// (angle, start) pairs: at 15 angles per wave and one pass it gives 3 to 10 %
// (80^3 S12 1.41 against 1.54 ms), at 12 it loses 2 %.
void pick_shape64(int nang, const rt_grid &g, long long ncell, KShape &k) {
  const long long tiles = (ncell + 63) / 64;
  const bool small = tiles <= 256;
  int slots = 0;
  if (nang <= 4) {
    slots = slots64_for(nang);
  } else if (small) {
    const int n = (nang + 15) / 16;
    slots = slots64_for(n < 2 ? 2 : n);
  } else {
    slots = slots64_for((nang + 3) / 4);
  }
  if (!slots || (nang + slots - 1) / slots > max_waves64(slots))
    slots = slots64_for((nang + 11) / 12);
  int waves = slots ? (nang + slots - 1) / slots : 0;
  if (!slots) {
    if (k.second) return;  // second order keeps its increments in registers
    slots = kStagedSlots;
    long long best = 1ll << 40;
    for (int w = max_waves64(slots); w >= 4; --w) {
      const int ch = (nang + w * slots - 1) / (w * slots);
      // the fewest chunks where one block a CU runs, else the fewest padding slots
      const long long cost = small ? ch * 64ll + w : (long long)ch * w;
      if (cost < best) {
        best = cost;
        waves = w;
        k.geo.chunks = ch;
      }
    }
  }
  k.waves = waves;
  k.geo.slots = slots;
  const int nx = g.n[0];
  const int starts = nx % 64 == 0 ? 1 : 1 + (62 + nx) / nx;
  k.geo.xs = nx >= 8 && slots >= kSharedSlots * ((slots * starts + 63) / 64);
}

long long cell_blocks(const rt_ctx *c) { return (c->ncell + kBlock - 1) / kBlock; }

bool fields_ok(const rt_fields *f) {
  return f && f->sigma_a && f->sigma_s && f->rho && f->T && f->v;
}

void launch_step(const rt_ctx *c, const StepArgs &a, bool fused, hipStream_t s) {
  clear_stale_error();
  if (c->p.precision == RT_FP32_MIXED)
    launch_step_f32(a, c->shape, fused, ctx_step_blocks(c, fused), s);
  else
    launch_step_f64(a, c->shape, fused, ctx_step_blocks(c, fused), s);
}

void launch_transport(const rt_ctx *c, const StepArgs &a, hipStream_t s) {
  clear_stale_error();
  dim3 g((unsigned)cell_blocks(c)), b(kBlock);
  if (c->p.precision == RT_FP32_MIXED) {
    if (c->all_periodic)
      hipLaunchKernelGGL((k_transport<float, float, true>), g, b, 0, s, a);
    else
      hipLaunchKernelGGL((k_transport<float, float, false>), g, b, 0, s, a);
  } else if (c->shape.waves) {
    launch_step64(a, c->shape, kTransportOnly64, ctx_step_blocks(c, true), s);
  } else {
    if (c->all_periodic)
      hipLaunchKernelGGL((k_transport<double, double, true>), g, b, 0, s, a);
    else
      hipLaunchKernelGGL((k_transport<double, double, false>), g, b, 0, s, a);
  }
}

void launch_moments(const rt_ctx *c, const StepArgs &a, hipStream_t s) {
  clear_stale_error();
  dim3 g((unsigned)cell_blocks(c)), b(kBlock);
  if (c->p.precision == RT_FP32_MIXED)
    hipLaunchKernelGGL(k_moments<float>, g, b, 0, s, a);
  else
    hipLaunchKernelGGL(k_moments<double>, g, b, 0, s, a);
}

int ensure_moments(rt_ctx *c, hipStream_t s) {
  if (c->mom_valid) return RT_OK;
  return ctx_moments(c, s);
}

hipEvent_t take_event(rt_ctx *c) {
  if (!c->ev_pool.empty()) {
    hipEvent_t e = c->ev_pool.back();
    c->ev_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// One step (fused or from a given dF); swaps the current buffers.
int one_step(rt_ctx *c, double dt, const rt_fields *f, const void *dF, bool fused, rt_out *o,
             bool first, bool last, hipStream_t s) {
  StepArgs a;
  ctx_fill_args(c, dt, f, a);
  a.I_in = c->I[c->cur];
  a.I_out = c->I[1 - c->cur];
  a.mom_in = c->mom[c->mom_cur];
  a.mom_out = c->mom[1 - c->mom_cur];
  a.dF_in = dF;
  a.nparts = (int)ctx_step_blocks(c, fused);
  a.accumulate = first ? 0 : 1;
  if (o) {
    a.dEgas = o->dEgas;
    a.dMom = o->dMom;
    if (last) {
      a.oE = o->Er;
      a.oF = o->Fr;
      a.oP = o->Pr;
    }
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (c->profile && fused) {
    e0 = take_event(c);
    e1 = take_event(c);
    if (e0 && e1) hipEventRecord(e0, s);
  }
  launch_step(c, a, fused, s);
  if (!hip_ok(hipGetLastError())) return RT_EDEVICE;
  if (e0 && e1) {
    hipEventRecord(e1, s);
    c->pending.emplace_back(e0, e1);
  }
  if (last && o && o->totals) {
    // chunk rows go into the interface table, which the last step has read
    const int nch = tot_chunks(a.nparts);
    double *dst = nch > 1 ? c->faces : o->totals;
    hipLaunchKernelGGL(k_totals, dim3((unsigned)nch), dim3(64 * kNtot), 0, s, c->partials,
                       a.nparts, dst);
    if (nch > 1)
      hipLaunchKernelGGL(k_totals_join, dim3(1), dim3(64 * kNtot), 0, s, c->faces, nch,
                         o->totals);
    if (!hip_ok(hipGetLastError())) return RT_EDEVICE;
  }
  c->cur = 1 - c->cur;
  c->mom_cur = 1 - c->mom_cur;
  c->mom_valid = true;
  return RT_OK;
}

}  // namespace

long long ctx_step_blocks(const rt_ctx *c, bool fused) {
  // the wave-group kernel works in tiles of 64 cells; a second-order step
  // from a given dF runs on the thread-per-cell kernel
  const bool tiles = c->shape.waves && (fused || !c->shape.second);
  return tiles ? (c->ncell + 63) / 64 : (c->ncell + kBlock - 1) / kBlock;
}

int ctx_storage_bytes(const rt_ctx *c) { return c->p.precision == RT_FP32_MIXED ? 4 : 8; }

// The speed at which the radiation advances: c, or the reduced speed.
double radiation_speed(const rt_ctx *c) {
  return c->p.c_reduced > 0.0 ? c->p.c_reduced : c->p.c;
}

int ctx_check_dt(const rt_ctx *c, double dt) {
  if (!(dt > 0.0) || !std::isfinite(dt)) return RT_EINVAL;
  if (radiation_speed(c) * dt * c->cfl_sum > 1.0 + 1e-12) return RT_ECFL;
  return RT_OK;
}

void ctx_fill_args(const rt_ctx *c, double dt_call, const rt_fields *f, StepArgs &a) {
  std::memset(&a, 0, sizeof(a));
  // with the reduced speed of light the radiation takes the step dt c_r/C in
  // every one of its terms (transport and sources); the gas keeps the true
  // coupling through a heat capacity (and, in the outputs, momentum) scaled
  // by c_r/C, which gives the temperature of the true-rate gas equation
  const double sc = radiation_speed(c) / c->p.c;
  const double dt = dt_call * sc;
  a.gasfac = 1.0 / sc;
  a.ndim = c->g.ndim;
  a.ivfac = (c->p.flags & RT_ORIGINAL_TRANSPORT) ? 0.0 : 3.0;
  for (int d = 0; d < 3; ++d) {
    a.n[d] = c->g.n[d];
    for (int s = 0; s < 2; ++s) a.bc[d][s] = c->g.bc[d][s];
    a.dt_dx[d] = dt / c->g.dx[d];
    // the original transport has alpha = 1 at every interface (zero length
    // scale in its optical depth) and no IV split (IV = 0, I~ = I)
    a.dl10[d] = (c->p.flags & RT_ORIGINAL_TRANSPORT) ? 0.0 : 10.0 * c->g.dx[d];
  }
  a.inv_n0 = 1.0 / c->g.n[0];
  a.inv_n1 = 1.0 / c->g.n[1];
  a.stride[0] = 1;
  a.stride[1] = c->g.n[0];
  a.stride[2] = c->g.n[0] * c->g.n[1];
  a.ncell = (int)c->ncell;
  a.nang = c->nang;
  a.dt = dt;
  a.C = c->p.c;
  a.invC = 1.0 / c->p.c;
  a.P = c->p.prat;
  a.cvfac = c->p.r_ideal / (c->p.gamma - 1.0) * sc;
  double vol = 1.0;
  for (int d = 0; d < c->g.ndim; ++d) vol *= c->g.dx[d];
  a.vol = vol;
  a.rtol = c->p.newton_rtol;
  a.maxit = c->p.newton_maxit;
  a.estimate_v = (c->p.flags & RT_ESTIMATE_V) ? 1 : 0;
  a.mu = c->d_mu;
  a.w = c->d_w;
  a.ghost = c->d_ghost;
  a.arec = c->d_arec;
  a.arecf = c->d_arecf;
  for (int k = 0; k < 10; ++k) a.wmom[k] = c->wmom[k];
  for (int f = 0; f < 6; ++f) a.gface[f] = c->d_gface[f];
  a.faces = c->faces;
  if (f) {
    a.sa = f->sigma_a;
    a.ss = f->sigma_s;
    a.rho = f->rho;
    a.v = f->v;
    a.feedback = (c->p.flags & RT_GAS_FEEDBACK) ? 1 : 0;
    a.T = f->T;
  }
  a.status = c->status;
  a.partials = c->partials;
  a.nparts = (int)ctx_step_blocks(c, true);
}

int ctx_init_host(const rt_grid *g, const rt_angles *an, const rt_params *p, rt_ctx *c) {
  if (!g || !an || !p) return RT_EINVAL;
  if (g->ndim < 1 || g->ndim > 3) return RT_EINVAL;
  long long nc = 1;
  for (int d = 0; d < 3; ++d) {
    if (g->n[d] < 1) return RT_EINVAL;
    if (d >= g->ndim && g->n[d] != 1) return RT_EINVAL;
    if (d < g->ndim) {
      if (!(g->dx[d] > 0.0) || !std::isfinite(g->dx[d])) return RT_EINVAL;
      for (int s = 0; s < 2; ++s)
        if (g->bc[d][s] < RT_BC_PERIODIC || g->bc[d][s] > RT_BC_VACUUM) return RT_EINVAL;
      if ((g->bc[d][0] == RT_BC_PERIODIC) != (g->bc[d][1] == RT_BC_PERIODIC)) return RT_EINVAL;
    }
    nc *= g->n[d];
  }
  if (nc > 0x7fffffffLL) return RT_EUNSUPPORTED;
  if (an->n < 1 || an->n > RT_MAX_ANGLES || !an->mu || !an->w) return RT_EINVAL;
  double wsum = 0.0;
  for (int m = 0; m < an->n; ++m) {
    const double *n = an->mu + 3 * m;
    const double nn = std::sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    // 1D slabs may use azimuthally averaged directions (mu, 0, 0), |n| <= 1
    const bool norm_ok = g->ndim == 1 ? nn <= 1.0 + 1e-12 : std::fabs(nn - 1.0) <= 1e-12;
    if (!norm_ok || !(an->w[m] > 0.0)) return RT_EBADQUAD;
    wsum += an->w[m];
  }
  if (!(std::fabs(wsum - 1.0) <= 1e-12)) return RT_EBADQUAD;
  if (!(p->c > 0.0) || !(p->prat >= 0.0) || !(p->gamma > 1.0) || !(p->r_ideal > 0.0))
    return RT_EINVAL;
  if (p->precision != RT_FP64 && p->precision != RT_FP32_MIXED) return RT_EINVAL;
  if (!(p->c_reduced >= 0.0) || p->c_reduced > p->c) return RT_EINVAL;
  if (p->c_reduced > 0.0 && p->c_reduced < p->c && (p->flags & RT_ESTIMATE_V))
    return RT_EUNSUPPORTED;
  const bool tiles = plane_fits(nc, p->precision == RT_FP32_MIXED ? 4 : 8);
  // the thread-per-cell kernels hold the velocity fixed
  if (!tiles && (p->flags & RT_GAS_FEEDBACK)) return RT_EUNSUPPORTED;

  c->g = *g;
  c->p = *p;
  if (!(c->p.newton_rtol > 0.0)) c->p.newton_rtol = 1e-14;
  if (c->p.newton_maxit <= 0) c->p.newton_maxit = 64;
  c->nang = an->n;
  c->ncell = nc;
  c->all_periodic = true;
  for (int d = 0; d < g->ndim; ++d)
    if (g->bc[d][0] != RT_BC_PERIODIC) c->all_periodic = false;
  const int N = an->n;
  c->h_mu.assign(3 * (size_t)N, 0.0);
  c->h_w.assign(an->w, an->w + N);
  c->h_ghost.assign(6 * (size_t)N, 0.0);
  c->cfl_sum = 0.0;
  for (double &x : c->wmom) x = 0.0;
  for (int m = 0; m < N; ++m) {
    const double *q = an->mu + 3 * m, w = an->w[m];
    const double b[10] = {1.0, q[0], q[1], q[2], q[0] * q[0], q[1] * q[1], q[2] * q[2],
                          q[0] * q[1], q[0] * q[2], q[1] * q[2]};
    for (int k = 0; k < 10; ++k) c->wmom[k] += w * b[k];
    double s = 0.0;
    for (int k = 0; k < 3; ++k) {
      c->h_mu[(size_t)k * N + m] = an->mu[3 * m + k];
      if (k < g->ndim) s += std::fabs(an->mu[3 * m + k]) / g->dx[k];
    }
    if (s > c->cfl_sum) c->cfl_sum = s;
  }
  c->shape = KShape();
  c->shape.periodic = c->all_periodic;
  // second order: the fused step runs both absorption solves on the
  // wave-group kernel; the step from a given dF on the thread-per-cell one
  c->shape.second = (p->flags & RT_SECOND_ORDER) != 0;
  if (tiles && p->precision == RT_FP32_MIXED)
    pick_shape32(N, c->shape);
  else if (tiles)
    pick_shape64(N, *g, nc, c->shape);
  c->nblocks = (nc + 63) / 64;  // enough partial-total rows for either kernel
  // angle records: every slot of the wave-group kernel has one (padding
  // slots a zero record)
  const int slots = p->precision == RT_FP32_MIXED
                        ? c->shape.waves * c->shape.groups * kAnglesPerWave
                        : c->shape.waves * c->shape.geo.slots * c->shape.geo.chunks;
  c->nrec = slots > N ? slots : N;
  return RT_OK;
}

namespace {
// Scratch layout: offsets of the pieces in one block.
struct Plan {
  size_t mu, w, ghost, arec, arecf, mom0, mom1, faces, partials, status, total;
};
Plan plan_of(const rt_ctx *c) {
  Plan q;
  const size_t N = c->nang, nc = c->ncell;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += align256(bytes);
    return at;
  };
  q.mu = take(sizeof(double) * 3 * N);
  q.w = take(sizeof(double) * N);
  q.ghost = take(sizeof(double) * 6 * N);
  q.arec = take(sizeof(double) * kRec * (size_t)c->nrec);
  q.arecf = take(c->p.precision == RT_FP32_MIXED ? sizeof(float) * kRec * (size_t)c->nrec : 0);
  q.mom0 = take(sizeof(double) * kNmomX * nc);
  q.mom1 = take(sizeof(double) * kNmomX * nc);
  q.faces = take(sizeof(double) * 9 * nc);
  q.partials = take(sizeof(double) * kNtot * c->nblocks);
  q.status = take(sizeof(int));
  q.total = o;
  return q;
}
}  // namespace

size_t ctx_scratch_bytes(const rt_ctx *c) { return plan_of(c).total; }
size_t ctx_table_bytes(const rt_ctx *c) { return plan_of(c).arec; }

int ctx_attach_scratch(rt_ctx *c, char *base, hipStream_t s, char *stage) {
  const Plan q = plan_of(c);
  const size_t N = c->nang;
  c->d_mu = reinterpret_cast<double *>(base + q.mu);
  c->d_w = reinterpret_cast<double *>(base + q.w);
  c->d_ghost = reinterpret_cast<double *>(base + q.ghost);
  c->d_arec = reinterpret_cast<double *>(base + q.arec);
  c->d_arecf = c->p.precision == RT_FP32_MIXED ? reinterpret_cast<float *>(base + q.arecf) : nullptr;
  c->mom[0] = reinterpret_cast<double *>(base + q.mom0);
  c->mom[1] = reinterpret_cast<double *>(base + q.mom1);
  c->faces = reinterpret_cast<double *>(base + q.faces);
  c->partials = reinterpret_cast<double *>(base + q.partials);
  c->status = reinterpret_cast<int *>(base + q.status);
  bool ok;
  if (stage) {  // the tables lie side by side: one copy
    std::memcpy(stage + q.mu, c->h_mu.data(), sizeof(double) * 3 * N);
    std::memcpy(stage + q.w, c->h_w.data(), sizeof(double) * N);
    std::memcpy(stage + q.ghost, c->h_ghost.data(), sizeof(double) * 6 * N);
    ok = hip_ok(hipMemcpyAsync(base, stage, q.arec, hipMemcpyHostToDevice, s));
  } else {
    ok = hip_ok(hipMemcpyAsync(c->d_mu, c->h_mu.data(), sizeof(double) * 3 * N,
                               hipMemcpyHostToDevice, s)) &&
         hip_ok(hipMemcpyAsync(c->d_w, c->h_w.data(), sizeof(double) * N, hipMemcpyHostToDevice,
                               s)) &&
         hip_ok(hipMemcpyAsync(c->d_ghost, c->h_ghost.data(), sizeof(double) * 6 * N,
                               hipMemcpyHostToDevice, s));
  }
  if (!ok) return RT_EDEVICE;
  clear_stale_error();
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, s, c->status, 0);
  return hip_ok(hipGetLastError()) ? RT_OK : RT_EDEVICE;
}

int ctx_moments(rt_ctx *c, hipStream_t s) {
  StepArgs a;
  ctx_fill_args(c, 1.0, nullptr, a);
  a.I_in = c->I[c->cur];
  a.mom_out = c->mom[c->mom_cur];
  launch_moments(c, a, s);
  if (!hip_ok(hipGetLastError())) return RT_EDEVICE;
  c->mom_valid = true;
  return RT_OK;
}

// Per-call tables: interface alpha / flow speed / IV Courant factor for this
// dt and fields, and 3 v J of the current moments.
int ctx_prepare_call(rt_ctx *c, double dt, const rt_fields *f, hipStream_t s) {
  StepArgs a;
  ctx_fill_args(c, dt, f, a);
  clear_stale_error();
  const long long nthreads = c->ncell > c->nrec ? c->ncell : c->nrec;
  hipLaunchKernelGGL(k_faces, dim3((unsigned)((nthreads + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                     s, a, c->faces, c->mom[c->mom_cur], c->d_arec, c->d_arecf, c->nrec);
  return hip_ok(hipGetLastError()) ? RT_OK : RT_EDEVICE;
}

int ctx_step(rt_ctx *c, double dt, int nsteps, const rt_fields *f, rt_out *o, hipStream_t s) {
  int st = ensure_moments(c, s);
  if (st != RT_OK) return st;
  st = ctx_prepare_call(c, dt, f, s);
  if (st != RT_OK) return st;
  return ctx_step_range(c, dt, f, o, 0, nsteps, nsteps, s);
}

int ctx_step_range(rt_ctx *c, double dt, const rt_fields *f, rt_out *o, int k0, int k1,
                   int ntotal, hipStream_t s) {
  const bool feedback = (c->p.flags & RT_GAS_FEEDBACK) != 0;
  for (int k = k0; k < k1; ++k) {
    // with gas feedback the flow speeds of the interface table follow v
    if (feedback && k > k0) {
      const int st = ctx_prepare_call(c, dt, f, s);
      if (st != RT_OK) return st;
    }
    const int st = one_step(c, dt, f, nullptr, true, o, k == 0, k == ntotal - 1, s);
    if (st != RT_OK) return st;
  }
  return RT_OK;
}

int ctx_init_equilibrium(rt_ctx *c, const double *T, void *I, hipStream_t s) {
  dim3 g((unsigned)cell_blocks(c)), b(kBlock);
  clear_stale_error();
  if (c->p.precision == RT_FP32_MIXED)
    hipLaunchKernelGGL(k_equilibrium<float>, g, b, 0, s, T, static_cast<float *>(I),
                       (int)c->ncell, c->nang);
  else
    hipLaunchKernelGGL(k_equilibrium<double>, g, b, 0, s, T, static_cast<double *>(I),
                       (int)c->ncell, c->nang);
  return hip_ok(hipGetLastError()) ? RT_OK : RT_EDEVICE;
}

}  // namespace rtk

// ------------------------------------------------------ static scratch
// The library scratch of rt_step_static: one array per GPU (each device that
// runs the library holds its own copy until the process ends).  Host code
// reaches it only through the device address that hipGetSymbolAddress gives
// for the current device, once per device, kept in static_ptr[]; the array's
// name is a host-side stand-in, not a device address.
static __device__ __align__(256) char scratch[RT_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kStaticDevices = 16;
std::mutex static_mu;
char *static_ptr[kStaticDevices];
// Host contexts of rt_step_static, one per device, with their host tables
// reserved for RT_MAX_ANGLES directions when the library loads, so that the
// calls themselves allocate nothing (the tables are refilled in place).
rt_ctx *static_ctx[kStaticDevices];

__attribute__((constructor)) void static_ctx_init() {
  for (int d = 0; d < kStaticDevices; ++d) {
    rt_ctx *c = new (std::nothrow) rt_ctx();
    if (!c) continue;
    const size_t N = RT_MAX_ANGLES;
    c->h_mu.reserve(3 * N);
    c->h_w.reserve(N);
    c->h_ghost.reserve(6 * N);
    static_ctx[d] = c;
  }
}
}  // namespace

using namespace rtk;

extern "C" {

int rt_step_static(const rt_grid *g, const rt_angles *an, const rt_params *p, void *Ia, void *Ib,
                   double dt, int nsteps, const rt_fields *f, rt_out *o, int *status,
                   void *stream) {
  if (!g || !an || !p || !Ia || !Ib || Ia == Ib || !fields_ok(f) || !status || nsteps < 0)
    return RT_EINVAL;
  int dev = -1;
  if (!hip_ok(hipGetDevice(&dev)) || dev < 0 || dev >= kStaticDevices) return RT_EDEVICE;
  char *base = nullptr;
  {
    std::lock_guard<std::mutex> lk(static_mu);
    if (!static_ptr[dev]) {
      void *ptr = nullptr;
      if (!hip_ok(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) || !ptr) {
        clear_stale_error();
        return RT_EDEVICE;
      }
      static_ptr[dev] = static_cast<char *>(ptr);
    }
    base = static_ptr[dev];
  }
  rt_ctx *c = static_ctx[dev];
  if (!c) return RT_ENOMEM;
  c->owns_device = false;
  c->profile = false;
  for (auto &t : c->d_gface) t = nullptr;
  int st = ctx_init_host(g, an, p, c);
  if (st != RT_OK) return st;
  if (ctx_scratch_bytes(c) > RT_STATIC_SCRATCH_BYTES) return RT_ETOOBIG;
  if ((c->p.flags & RT_GAS_FEEDBACK) && c->nang > kMaxFeedbackAngles) return RT_EUNSUPPORTED;
  st = ctx_check_dt(c, dt);
  if (st != RT_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  st = ctx_attach_scratch(c, base, s);
  if (st != RT_OK) return st;
  c->status = status;  // the caller's flag
  c->I[0] = Ia;
  c->I[1] = Ib;
  c->cur = 0;
  c->mom_cur = 0;
  c->mom_valid = false;
  return ctx_step(c, dt, nsteps, f, o, s);
}


const char *rt_strerror(int st) {
  switch (st) {
    case RT_OK: return "ok";
    case RT_PENDING: return "request still in flight";
    case RT_EINVAL: return "invalid argument";
    case RT_ENOMEM: return "out of memory";
    case RT_EDEVICE: return "HIP runtime error";
    case RT_ECFL: return "time step violates the transport CFL limit";
    case RT_ENOCONV: return "temperature Newton iteration failed";
    case RT_EBADQUAD: return "invalid angle set (weights or direction norms)";
    case RT_ESTATE: return "call order violated (no intensity bound?)";
    case RT_EUNSUPPORTED: return "unsupported request";
    case RT_ETOOBIG: return "problem scratch exceeds the static scratch array";
    default: return "unknown status";
  }
}

int rt_create(const rt_grid *g, const rt_angles *an, const rt_params *p, rt_ctx **out) {
  if (!out) return RT_EINVAL;
  *out = nullptr;
  rt_ctx *c = new (std::nothrow) rt_ctx();
  if (!c) return RT_ENOMEM;
  int st = ctx_init_host(g, an, p, c);
  if (st != RT_OK) {
    delete c;
    return st;
  }
  hipGetDevice(&c->device);
  char *base = nullptr;
  if (!hip_ok(hipMalloc(&base, ctx_scratch_bytes(c)))) {
    delete c;
    return RT_ENOMEM;
  }
  c->owns_device = true;
  st = ctx_attach_scratch(c, base, nullptr);
  if (st == RT_OK && !hip_ok(hipStreamSynchronize(nullptr))) st = RT_EDEVICE;
  if (st != RT_OK) {
    rt_destroy(c);
    return st;
  }
  *out = c;
  return RT_OK;
}

int rt_destroy(rt_ctx *c) {
  if (!c) return RT_EINVAL;
  hipDeviceSynchronize();
  // the scratch block starts at the angle table
  if (c->owns_device && c->d_mu) hipFree(c->d_mu);
  for (auto f : c->d_gface)
    if (f) hipFree(f);
  for (auto &pr : c->pending) {
    hipEventDestroy(pr.first);
    hipEventDestroy(pr.second);
  }
  for (auto e : c->ev_pool) hipEventDestroy(e);
  delete c;
  return RT_OK;
}

int rt_bind_intensity(rt_ctx *c, void *Ia, void *Ib) {
  if (!c || !Ia || !Ib || Ia == Ib) return RT_EINVAL;
  c->I[0] = Ia;
  c->I[1] = Ib;
  c->cur = 0;
  c->mom_valid = false;
  return RT_OK;
}

int rt_current_intensity(rt_ctx *c, void **cur) {
  if (!c || !cur) return RT_EINVAL;
  if (!c->I[0]) return RT_ESTATE;
  *cur = c->I[c->cur];
  return RT_OK;
}

int rt_set_fixed_bc(rt_ctx *c, int axis, int side, const double *tab) {
  if (!c || !tab || axis < 0 || axis >= c->g.ndim || side < 0 || side > 1) return RT_EINVAL;
  if (c->g.bc[axis][side] != RT_BC_FIXED) return RT_EINVAL;
  const int f = axis * 2 + side;
  const size_t off = (size_t)f * c->nang;
  std::memcpy(&c->h_ghost[off], tab, sizeof(double) * c->nang);
  // steps queued on a caller's stream may still read the table: the upload
  // waits for them (the null-stream copy alone does not order against
  // non-blocking streams)
  if (!hip_ok(hipDeviceSynchronize())) return RT_EDEVICE;
  if (!hip_ok(hipMemcpy(c->d_ghost + off, tab, sizeof(double) * c->nang, hipMemcpyHostToDevice)))
    return RT_EDEVICE;
  // the angle table replaces a position-dependent one
  if (c->d_gface[f]) {
    hipFree(c->d_gface[f]);
    c->d_gface[f] = nullptr;
  }
  return RT_OK;
}

int rt_set_fixed_bc_face(rt_ctx *c, int axis, int side, const double *tab) {
  if (!c || !tab || axis < 0 || axis >= c->g.ndim || side < 0 || side > 1) return RT_EINVAL;
  if (c->g.bc[axis][side] != RT_BC_FIXED || !c->owns_device) return RT_EINVAL;
  const int f = axis * 2 + side;
  const size_t n = (size_t)c->nang * (size_t)(c->ncell / c->g.n[axis]);
  if (!c->d_gface[f]) {
    if (hipMalloc(&c->d_gface[f], sizeof(double) * n) != hipSuccess) {
      c->d_gface[f] = nullptr;
      clear_stale_error();
      return RT_ENOMEM;
    }
  } else {
    hipDeviceSynchronize();  // a step in flight may still read the table
  }
  if (!hip_ok(hipMemcpy(c->d_gface[f], tab, sizeof(double) * n, hipMemcpyHostToDevice)))
    return RT_EDEVICE;
  return RT_OK;
}

int rt_moments(rt_ctx *c, rt_out *o, void *stream) {
  if (!c) return RT_EINVAL;
  if (!c->I[0]) return RT_ESTATE;
  hipStream_t s = (hipStream_t)stream;
  StepArgs a;
  ctx_fill_args(c, 1.0, nullptr, a);
  a.I_in = c->I[c->cur];
  a.mom_out = c->mom[c->mom_cur];
  if (o) {
    a.oE = o->Er;
    a.oF = o->Fr;
    a.oP = o->Pr;
  }
  launch_moments(c, a, s);
  if (!hip_ok(hipGetLastError())) return RT_EDEVICE;
  c->mom_valid = true;
  return RT_OK;
}

int rt_transport(rt_ctx *c, double dt, const rt_fields *f, void *dF, void *stream) {
  if (!c || !dF || !fields_ok(f)) return RT_EINVAL;
  if (!c->I[0]) return RT_ESTATE;
  int st = ctx_check_dt(c, dt);
  if (st != RT_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  st = ensure_moments(c, s);
  if (st != RT_OK) return st;
  st = ctx_prepare_call(c, dt, f, s);
  if (st != RT_OK) return st;
  StepArgs a;
  ctx_fill_args(c, dt, f, a);
  a.I_in = c->I[c->cur];
  a.mom_in = c->mom[c->mom_cur];
  a.dF_out = dF;
  launch_transport(c, a, s);
  return hip_ok(hipGetLastError()) ? RT_OK : RT_EDEVICE;
}

int rt_source_implicit(rt_ctx *c, double dt, const rt_fields *f, const void *dF, rt_out *o,
                       void *stream) {
  if (!c || !fields_ok(f)) return RT_EINVAL;
  if (!c->I[0]) return RT_ESTATE;
  if ((c->p.flags & RT_GAS_FEEDBACK) && c->nang > kMaxFeedbackAngles) return RT_EUNSUPPORTED;
  // the second-order step from a given dF runs per cell, without feedback
  if ((c->p.flags & RT_GAS_FEEDBACK) && c->shape.second) return RT_EUNSUPPORTED;
  if (!(dt > 0.0) || !std::isfinite(dt)) return RT_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  int st = ensure_moments(c, s);
  if (st != RT_OK) return st;
  st = ctx_prepare_call(c, dt, f, s);
  if (st != RT_OK) return st;
  return one_step(c, dt, f, dF, false, o, true, true, s);
}

int rt_step(rt_ctx *c, double dt, int nsteps, const rt_fields *f, rt_out *o, void *stream) {
  if (!c || !fields_ok(f) || nsteps < 0) return RT_EINVAL;
  if (!c->I[0]) return RT_ESTATE;
  if ((c->p.flags & RT_GAS_FEEDBACK) && c->nang > kMaxFeedbackAngles) return RT_EUNSUPPORTED;
  int st = ctx_check_dt(c, dt);
  if (st != RT_OK) return st;
  return ctx_step(c, dt, nsteps, f, o, (hipStream_t)stream);
}

int rt_equilibrium_intensity(rt_ctx *c, const double *T, void *I, void *stream) {
  if (!c || !T || !I) return RT_EINVAL;
  if (I == c->I[c->cur]) c->mom_valid = false;
  return ctx_init_equilibrium(c, T, I, (hipStream_t)stream);
}

int rt_sync_status(rt_ctx *c) {
  if (!c) return RT_EINVAL;
  if (!hip_ok(hipDeviceSynchronize())) return RT_EDEVICE;
  int h = 0;
  if (!hip_ok(hipMemcpy(&h, c->status, sizeof(int), hipMemcpyDeviceToHost))) return RT_EDEVICE;
  if (h) {
    hipMemset(c->status, 0, sizeof(int));
    return RT_ENOCONV;
  }
  return RT_OK;
}

int rt_profile_enable(rt_ctx *c, int enable) {
  if (!c) return RT_EINVAL;
  c->profile = enable != 0;
  return RT_OK;
}

int rt_profile_read(rt_ctx *c, double *total_ms, int *launches) {
  if (!c) return RT_EINVAL;
  for (auto &pr : c->pending) {
    if (!hip_ok(hipEventSynchronize(pr.second))) return RT_EDEVICE;
    float ms = 0.f;
    if (!hip_ok(hipEventElapsedTime(&ms, pr.first, pr.second))) return RT_EDEVICE;
    c->prof_ms += ms;
    c->prof_n += 1;
    c->ev_pool.push_back(pr.first);
    c->ev_pool.push_back(pr.second);
  }
  c->pending.clear();
  if (total_ms) *total_ms = c->prof_ms;
  if (launches) *launches = c->prof_n;
  c->prof_ms = 0.0;
  c->prof_n = 0;
  return RT_OK;
}

int rt_get_info(rt_ctx *c, rt_info *info) {
  if (!c || !info) return RT_EINVAL;
  info->nang = c->nang;
  info->ncell = c->ncell;
  info->storage_bytes = ctx_storage_bytes(c);
  info->block_threads = c->shape.waves ? 64 * c->shape.waves : kBlock;
  info->grid_blocks = ctx_step_blocks(c, true);
  return RT_OK;
}

}  // extern "C"
