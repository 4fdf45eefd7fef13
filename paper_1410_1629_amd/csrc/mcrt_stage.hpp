// mcrt_stage.hpp -- the life cycle cut into stages: the per-lane logic of the
// kernels that large runs use (k_emit, k_leg, k_event).
//
// Method: Camps & Baes (arXiv:1410.1629), as mcrt_lane.hpp: the same draws,
// walks and estimators in the same order of arithmetic, so a package's
// history is the same to the bit.
//
// mcrt_lane.hpp keeps a package in one lane from emission to its end, and a
// wavefront alternates between the walk and the events of the lanes that
// wait: every event pass runs with a part of the lanes, and the kernel holds
// the walk's and the events' registers together.  Here all packages of a
// chunk advance together, one scattering order at a time.  Their state lies
// in memory in between (StagePkg, dense lists):
//   k_emit   emission, the peel-off rays of the emission: list 0;
//   k_move   order n: the list in the order of the packages' places;
//   k_leg    order n: walks each package's leg to the boundary for its
//            optical depth T, draws the forced-scattering depth and walks to
//            that point: T and the length s per package;
//   k_event  order n: moves every package to its interaction point, peels
//            off, ends it or turns it: list n + 1.
// The walks run in a lean kernel, the events with every lane busy, and the
// state costs some 400 bytes of streaming per leg.  Once a list is short the
// walks' latency is all that is left, and the lane machine takes the rest of
// its packages' lives (lane_events with an accessor that resumes).
//
// Events in order of place also queue their peel rays so: the queue's walks
// then find neighbouring rays' records in one place.
#pragma once

#include "mcrt_lane.hpp"

namespace mcrt {

// What a stage kernel does: the forward run, or the adjoint's pass A.
enum StagePass : int { kPassForward = 0, kPassA = 1 };

// A leg's optical depth and the length to the next event.
struct alignas(16) StageLeg {
  double T, s;
};

// The position key of a package: the model box halved kStageKeyBits times,
// each time along its longest side (axis[l], two bits each), which numbers
// compact regions in Morton order.
constexpr int kStageKeyBits = 12;
struct StageKeys {
  unsigned axis;
  int bits[3];
  double lo[3], scale[3];
};

MCRT_HD unsigned stage_key(const StageKeys& K, const double r[3]) {
  unsigned c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double top = (double)((1 << K.bits[a]) - 1);
    c[a] = (unsigned)fmin(fmax((r[a] - K.lo[a]) * K.scale[a], 0.0), top) << (31 & (32 - K.bits[a]));
    if (K.bits[a] == 0) c[a] = 0;
  }
  unsigned key = 0;
  for (int l = 0; l < kStageKeyBits; ++l) {
    const unsigned a = (K.axis >> (2 * l)) & 3u;
    const unsigned bit = (a == 0 ? c[0] : (a == 1 ? c[1] : c[2])) >> 31;
    key = (key << 1) | bit;
    c[0] <<= a == 0;
    c[1] <<= a == 1;
    c[2] <<= a == 2;
  }
  return key;
}

inline StageKeys stage_keys(const GridDev& G) {
  StageKeys K;
  K.axis = 0;
  double side[3];
  for (int a = 0; a < 3; ++a) {
    K.bits[a] = 0;
    side[a] = G.hi[a] - G.lo[a];
  }
  for (int l = 0; l < kStageKeyBits; ++l) {
    const int a = side[0] >= side[1] ? (side[0] >= side[2] ? 0 : 2) : (side[1] >= side[2] ? 1 : 2);
    K.axis |= (unsigned)a << (2 * l);
    ++K.bits[a];
    side[a] *= 0.5;
  }
  for (int a = 0; a < 3; ++a) {
    K.lo[a] = G.lo[a];
    K.scale[a] = (double)(1 << K.bits[a]) / (G.hi[a] - G.lo[a]);
  }
  return K;
}

constexpr int kXcds = 8;  // a list is cut into one slice per XCD

struct StageParams {
  RunParams P;
  StageKeys K;
  const StagePkg* in;              // k_leg, k_event: the ordered list
  StageLeg* leg;                   // its packages' legs
  StagePkg* out;                   // k_emit, k_event: the next list and its position keys
  unsigned* keys;
  const unsigned long long* n_in;  // packages of `in`
  unsigned long long* n_out;       // packages appended to `out`
  unsigned long long* next;        // k_leg's next packages, one counter per slice
  unsigned long long min_n;        // lists shorter than this are left to the lane machine
  int n;                           // the order: events so far beyond the emission
};

MCRT_HD unsigned long long stage_package(const RunParams& P, unsigned slot, unsigned lam) {
  return P.first + (P.item0 + slot - (unsigned long long)lam * P.n_pkg);
}

// ---------------------------------------------------------------------------
// Legs.

// What a leg's walk is doing: the path to the boundary, the search for
// tau_s, or (rare) a second search for the end of the last absorbing segment
// of a leg whose tau_s rounding left beyond the first one's total.
enum LegMode : int { kLegPath = 0, kLegLocate, kLegLast };

template <typename R>
struct Leg {
  Ray<R, double> ry;
  int mode;
  bool found;
  unsigned slot, lam;
  double T, tau_s;
  R kapR;
  R tau_sR;  // kLegPath, kLegLast: +inf
  R comp, tau_prev, rho_hit;
  double last;  // kLegLast: end time of the last absorbing segment so far
};

template <typename R>
MCRT_HD void leg_init(Leg<R>& L) {
  L.ry.active = false;
  L.mode = kLegPath;
  L.slot = L.lam = 0;
  L.T = L.tau_s = 0.0;
  L.kapR = R(0);
}

// Back to the start of the walk: the indices step back by the planes
// crossed, the plane times stay.  (A tree walk keeps its point and leaf, so
// it is set up again.)
template <typename R, int GK>
MCRT_HD void leg_restart(Leg<R>& L, const GridDev& G, const double r[3], const double k[3]) {
  Ray<R, double>& ry = L.ry;
  if constexpr (GK == kGridTree) {
    ray_begin<R, GK>(ry, G, r, k);
  } else {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      ry.i[a] -= (int)ry.j[a] * ry.s[a];
      ry.j[a] = 0;
    }
    if constexpr (GK == kGridRect) {
#pragma unroll
      for (int a = 0; a < 3; ++a) ry.tp[a] = rect_tplane(ry, G, a);
    }
    ry.t = 0.0;
    ry.tau = R(0);
    ry.active = true;
  }
  L.comp = R(0);
}

// One block of crossings of the lane's walk, with lane_step's sums.  Every
// sub-step is evaluated (past b.n: the last end time again, no length)
// before the search ends, so that the block's density loads stay in flight
// together; the block that holds the point is gone through again.  Returns the positive-length crossings.
template <typename R, class Mem>
MCRT_HD unsigned leg_step(Leg<R>& L, const GridDev& G, Mem& M) {
  constexpr int D = kBlockWalk;
  Ray<R, double>& ry = L.ry;
  const R kapR = L.kapR;
  WalkBlock<D, R, double> b;
  ray_next_block(ry, b, G, M);
  bool hit = false;
  double t_run = ry.t;
  R run = ry.tau, comp = L.comp;
  unsigned n = 0;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const R s0 = (R)(b.tend[d] - t_run);  // one rounding of an FP64 difference
    const bool pos = s0 > R(0);
    const R dtau = kapR * b.rho[d] * (pos ? s0 : R(0));
    hit = hit || (pos && run + dtau > L.tau_sR);
    if (L.mode == kLegLast && dtau > R(0)) L.last = b.tend[d];
    if constexpr (sizeof(R) == sizeof(float)) {
      if (d < b.n) {  // compensated (Kahan), as lane_step
        const R y = dtau - comp;
        const R t = run + y;
        comp = (t - run) - y;
        run = t;
      }
    } else {
      run = d < b.n ? run + dtau : run;  // past the walk's end dtau is 0, or NaN in a cell of infinite density
    }
    n += pos;
    t_run = pos ? b.tend[d] : t_run;
  }
  if (!hit) {
    ry.tau = run;
    L.comp = comp;
    ry.t = t_run;
    if (b.out) ry.active = false;
    return n;
  }
  run = ry.tau;
  comp = L.comp;
  t_run = ry.t;
  n = 0;
  bool at = false;
  int dh = 0;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const R s0 = (R)(b.tend[d] - t_run);
    const bool pos = s0 > R(0);
    const R dtau = kapR * b.rho[d] * (pos ? s0 : R(0));
    if (!at) {
      n += pos;
      at = pos && run + dtau > L.tau_sR;
      if (at) {
        dh = d;
        L.rho_hit = b.rho[d];
        L.tau_prev = run;
      } else {
        if constexpr (sizeof(R) == sizeof(float)) {
          const R y = dtau - comp;
          const R t = run + y;
          comp = (t - run) - y;
          run = t;
        } else {
          run += dtau;
        }
        t_run = pos ? b.tend[d] : t_run;
      }
    }
  }
  L.found = true;
  ray_rewind<D, R, Mem::kGrid>(ry, b, dh, G);
  ry.active = false;
  return n;
}

// The forced-scattering depth of a leg of optical depth T after event n.
MCRT_HD double forced_depth(const RunParams& P, unsigned slot, unsigned lam, int n, double T) {
  const U4 ws = draw_words(P.seed, stage_package(P, slot, lam), lam, 2u + (unsigned)n);
  return -log1p(u01(ws.x) * expm1(-T));
}

// Takes package p: its path walk starts (one that misses the grid ends at once).
template <typename R, int GK, class Mem>
MCRT_HD void leg_begin(Leg<R>& L, const GridDev& G, Mem& M, const StagePkg& p) {
  L.slot = p.slot;
  L.lam = p.lam;
  L.kapR = (R)M.lam((int)p.lam).kappa;
  L.mode = kLegPath;
  L.found = false;
  L.tau_sR = R(INFINITY);
  L.comp = R(0);
  ray_begin<R, GK>(L.ry, G, p.r, p.k);
}

// The end of a walk of package p's leg after event n: the next walk is set
// up, or the leg is done and `out` its result (true).
template <typename R, int GK, class Mem>
MCRT_HD bool leg_end(Leg<R>& L, const RunParams& P, Mem& M, int n, const StagePkg& p, StageLeg& out) {
  if (L.mode == kLegPath) {
    L.T = (double)L.ry.tau;
    if (L.T == 0.0) {  // nothing to interact with: the package leaves
      out = StageLeg{0.0, 0.0};
      return true;
    }
    L.tau_s = forced_depth(P, L.slot, L.lam, n, L.T);
    L.tau_sR = (R)L.tau_s;
    L.found = false;
    L.mode = kLegLocate;
    leg_restart<R, GK>(L, P.G, p.r, p.k);
    return false;
  }
  if (L.found || L.mode == kLegLast) {  // the interaction point
    double s = L.ry.tin + L.last;
    if (L.found)
      s = ray_cell_entry64<R, GK>(L.ry, P.G, p.r, p.k) +
          (L.tau_s - (double)L.tau_prev) / (M.lam((int)L.lam).kappa * (double)L.rho_hit);
    out = StageLeg{L.T, s};
    return true;
  }
  L.mode = kLegLast;  // tau_s reached the total by rounding
  L.tau_sR = R(INFINITY);
  L.last = 0.0;
  leg_restart<R, GK>(L, P.G, p.r, p.k);
  return false;
}

// ---------------------------------------------------------------------------
// Events.

// A peel ray walked on the spot (the queue is full), as the lane machine
// walks it: FP64 times, compensated FP32 sums.  DEP: deposits fac l instead.
template <typename R, bool DEP, class Mem>
MCRT_HD R stage_peel_walk(const GridDev& G, Mem& M, const double r[3], const double kd[3], double tmax, R kapR,
                          double fac, unsigned long long& nx) {
  Ray<R, double> ry;
  ray_begin<R, Mem::kGrid>(ry, G, r, kd, tmax);
  R comp = R(0);
  while (ry.active) {
    WalkBlock<kBlockWalk, R, double> b;
    ray_next_block<kBlockWalk, R, Mem, !DEP>(ry, b, G, M);
#pragma unroll
    for (int d = 0; d < kBlockWalk; ++d) {
      if (d >= b.n) break;
      const double tm = (Mem::kInst && b.tend[d] > ry.tmax) ? ry.tmax : b.tend[d];
      const R s0 = (R)(tm - ry.t);
      const bool pos = s0 > R(0);
      nx += pos;
      if (DEP) {
        if (pos) M.add_grad(b.cell[d], fac * (double)s0);
      } else {
        const R dtau = kapR * b.rho[d] * (pos ? s0 : R(0));
        if constexpr (sizeof(R) == sizeof(float)) {
          const R y = dtau - comp;
          const R t = ry.tau + y;
          comp = (t - ry.tau) - y;
          ry.tau = t;
        } else {
          ry.tau += dtau;
        }
      }
      if (pos) ry.t = tm;
    }
    if (b.out || (Mem::kInst && ry.t >= ry.tmax)) ry.active = false;
  }
  return ry.tau;
}

// Counts and luminosities of one lane of k_emit or k_event.
struct StageCounts {
  double s_abs = 0.0, s_esc = 0.0, s_trunc = 0.0;
  unsigned long long x_peel = 0, n_ev = 0, n_pk = 0, n_pl = 0, n_dep = 0;
};

// Frames (one bit each) that event n at r projects into: its peel rays.
template <class Mem>
MCRT_HD unsigned stage_frames(const RunParams& P, Mem& M, int n, const double r[3]) {
  if (!(P.flags & (n == 0 ? kFlagPeelEmit : kFlagPeelScat))) return 0u;
  unsigned mask = 0;
  for (int d = 0; d < P.n_det; ++d)
    if (frame_pixel<Mem::kInst>(M.det(d), r) >= 0) mask |= 1u << d;
  return mask;
}

// Queues the peel rays of event n at r (incoming direction k, weight W
// there) towards the frames of `mask`, from queue slot `at` on; rays beyond
// the queue's capacity are walked here.
template <typename R, int PASS, class Mem>
MCRT_HD void stage_peel(const RunParams& P, Mem& M, int n, const double r[3], const double k[3], double W,
                        unsigned slot, unsigned lam, const LamDev& O, unsigned mask, unsigned long long at,
                        StageCounts& c) {
  const int comp = ((P.flags & kFlagSplit) && n > 0) ? 1 : 0;
  for (int d = 0; d < P.n_det; ++d) {
    if (!((mask >> d) & 1u)) continue;
    const DetDev& D = M.det(d);
    const int pix = frame_pixel<Mem::kInst>(D, r);
    const long long ii = ((long long)comp * P.n_lambda + lam) * P.pix_lambda + D.off + pix;
    const unsigned long long js = at++;
    const bool room = P.jobs && js < P.job_cap;
    double kd[3], inv_d2, tmax;
    peel_geom<Mem>(D, r, kd, inv_d2, tmax);
    const double ph = n == 0 ? 1.0 / (4.0 * kPi) : hg_phase(O.g, k[0] * kd[0] + k[1] * kd[1] + k[2] * kd[2]);
    const double v = W * ph * inv_d2;
    ++c.n_pl;
    if (room) {
      const int kp = key_pixel<Mem::kInst>(D, r, pix);
      M.store_job(js, r, v, ii, tile_key(D, kp), sort_sub(D, kp, r, P.depth_drop), slot,
                  n < kEventSat ? n : kEventSat, d, lam);
      continue;
    }
    const double tau = (double)stage_peel_walk<R, false>(P.G, M, r, kd, tmax, (R)O.kappa, 0.0, c.x_peel);
    const double C = W * ph * exp(-tau) * inv_d2;
    if (PASS == kPassForward) {
      M.add_image(ii, C);
      if (P.tape) M.tape_peel((int)slot, n, d, C, ii);
    } else {
      const double q = M.adj(ii) * C;
      M.ev_store((int)slot, n, 1 + d, q);
      if (q != 0.0) {
        unsigned long long nx = 0;
        stage_peel_walk<R, true>(P.G, M, r, kd, tmax, (R)O.kappa, -q * O.kappa, nx);
        c.x_peel += nx;
        c.n_dep += nx;
      }
    }
  }
}

// Emission of chunk item `slot`; false: the package is not born (nothing is
// emitted at its wavelength).
template <class Mem>
MCRT_HD bool stage_emit(const RunParams& P, Mem& M, unsigned slot, unsigned& lam, double r[3], double k[3],
                        double& W) {
  const unsigned long long item = P.item0 + slot;
  lam = P.n_lambda == 1 ? 0u : (unsigned)(item / P.n_pkg);
  const unsigned long long pkg = stage_package(P, slot, lam);
  const LamDev& LD = M.lam((int)lam);
  if (LD.ltot == 0.0) return false;
  const U4 wd = draw_words(P.seed, pkg, lam, 1u);
  int s = P.n_src - 1;
  const double target = u01(wd.z) * LD.ltot;
  for (int q = 0; q < P.n_src; ++q) {
    if (target < LD.cum[q]) {
      s = q;
      break;
    }
  }
  iso_direction(u01(wd.x), u01(wd.y), k);
  const SrcDev& src = M.src(s);
  const U4 wp = draw_words(P.seed, pkg, lam, 0u);
  if (src.kind == 2)
    cell_source_position<Mem::kGrid>(src, P.G, (int)lam, wp, r);
  else
    source_position(src, wp, r);
  W = LD.w0;
  return true;
}

// The event at the end of a leg of optical depth T and length s: the
// package moves there and its weight is updated; false: it left the grid.
template <int PASS, class Mem>
MCRT_HD bool stage_move(const RunParams& P, Mem& M, const LamDev& O, unsigned slot, int n, double T, double s,
                        double r[3], const double k[3], double& W, StageCounts& c) {
  if (PASS == kPassA) M.ev_store((int)slot, n, 0, T);
  if (PASS == kPassForward && P.tape) M.tape_leg((int)slot, n, T);
  if (T == 0.0) {
    c.s_esc += W;
    return false;
  }
  const double em = -expm1(-T);
  // the leg's absorbed fraction telescopes to 1 - e^-T (the forward's statistic alone: no tally here)
  if (PASS == kPassForward) c.s_abs += W * (1.0 - O.albedo) * em;
  c.s_esc += W * exp(-T);
  ++c.n_ev;
  r[0] += s * k[0];
  r[1] += s * k[1];
  r[2] += s * k[2];
  W *= O.albedo * em;
  return true;
}

// Whether the package ends with event n (weight W after it).
MCRT_HD bool stage_ends(const RunParams& P, const LamDev& O, int n, double W) {
  return W < P.w_min * O.w0 || n >= P.max_scatter;
}

// The direction after event n + 1, from the HG phase function.
MCRT_HD void stage_turn(const RunParams& P, const LamDev& O, unsigned slot, unsigned lam, int n, double k[3]) {
  const U4 ws = draw_words(P.seed, stage_package(P, slot, lam), lam, 2u + (unsigned)n);
  turn(k, hg_sample_mu(O.g, u01(ws.y)), u01(ws.z));
}

}  // namespace mcrt
