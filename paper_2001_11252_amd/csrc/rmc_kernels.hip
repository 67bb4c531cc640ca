// rmc_kernels.hip -- gfx950 kernels of the resonant-line Monte Carlo path.
//
// k_transport   persistent per-packet propagation loop (Sect. 3, 3.2, 4.3)
//               with peel-off toward observers at each emission and
//               scattering (Sect. 5.1); one packet per lane, lanes of a
//               wave refilled from the wave's reserve of a global queue
//               (ballot + mbcnt ranks of the idle lanes).  Each
//               peel-off ray is decided in the scattering's own leaf or
//               queued in the wave's region of the peel-off queue.
// k_walkers     the transport of a run's last packets: a few packets a wave,
//               their draws and peel-off computed by all its lanes
// k_peel_drain  ray-cast pass over the queued peel-off rays after each
//               transport launch (lanes refilled per ray), k_peel_scan
//               the index of its jobs
// k_trace       deterministic cell sequence of rays (probe)
// k_tau         optical depth of rays to the domain border (probe)
// k_image_fwd   peel-off image of fixed rays
// k_image_bwd   its adjoint with respect to per-leaf n_HI, kappa_d, v_los
// k_hist        spectrum of escaped packets
#include <mutex>

#include "rmc_device.h"
#include "rmc_launch.h"

namespace rmc {

// exp(-tau) is exactly zero (round to nearest) from these optical depths
// on: a ray may stop integrating there without changing any deposit.
template <class R> struct TauCut;
template <> struct TauCut<double> { static constexpr double v = 746.0; };
template <> struct TauCut<float> { static constexpr double v = 104.0; };

__device__ __forceinline__ void atomic_add_real(float *p, float v) { unsafeAtomicAdd(p, v); }
__device__ __forceinline__ void atomic_add_real(double *p, double v) { unsafeAtomicAdd(p, v); }

// --------------------------------------------------------------- ray cast
// A point strictly inside a cell is located in that cell whatever the
// direction, so a ray starting there needs no descent from the root.
__device__ __forceinline__ bool strictly_inside(const Cell &c, int L, const double p[3]) {
  const double inv = ldexp(1.0, -L);
  const int s = 1 << (L - c.level);
  const int o[3] = {c.ox, c.oy, c.oz};
  bool in = true;
#pragma unroll
  for (int d = 0; d < 3; ++d) in = in && (p[d] > (double)o[d] * inv) && (p[d] < (double)(o[d] + s) * inv);
  return in;
}

// Where a peel-off ray may start: the packet's current cell, its leaf
// record and the LDS stack of its ancestors.
template <class R> struct StartCell {
  const Cell *c;
  const LeafRec<R> *lf;
  const int *stk;
};

// Walks a ray at fixed x_ext from p (inside cell c) leaf by leaf, adding
// kappa * segment to tau, until it reaches the domain border or tau >=
// tau_cut.  steps counts the leaves crossed so far (at most MAX_CROSS).  With
// borrowed, sc lends the first leaf's record and ancestor stack.
template <class R, int NL>
__device__ double ray_walk(const ProblemK &pb, double p[3], const double k[3], double x_ext, double tau,
                           uint32_t steps, double tau_cut, int *stk, int stride, uint32_t *ncross, Cell &c,
                           const StartCell<R> *sc, bool borrowed, const double *kinv = nullptr) {
  const R kr[3] = {(R)k[0], (R)k[1], (R)k[2]};
  bool first = borrowed;
  bool start = true;
  for (; steps < MAX_CROSS; ++steps) {
    const LeafRec<R> lf = first ? *sc->lf : load_leaf<R>(pb.leaves, c.leaf);
    Opac<R, NL> o;
    opacity(pb, lf, x_ext, kr, o);
    // Only the start point can lie inside a leaf: later leaves are entered
    // on a face (inner distance 0, where the test is tau >= tau_cut, which
    // the previous leaf already ruled out).
    if (start && lf.bnd == R(0)) {
      if (tau + (double)o.ktot * inner_dist(c, pb.L, p) >= tau_cut) {
        // the cut is reached inside this leaf whatever the exit distance
        ++*ncross;
        tau = tau_cut;
        break;
      }
    }
    start = false;
    double face[3], lo[3], hi[3];
    int em;
    const double te = exit_dist(c, pb.L, p, k, face, lo, hi, &em, kinv);
    const double td = domain_dist_leaf(lf, pb.domain, pb.dom, p, k);
    ++*ncross;
    if (td <= te) {
      tau += (double)o.ktot * td;
      break;
    }
    tau += (double)o.ktot * te;
    if (tau >= tau_cut) break;
    double pn[3];
    exit_point(te, em, p, k, face, lo, hi, pn);
    p[0] = pn[0]; p[1] = pn[1]; p[2] = pn[2];
    wrap_slab(pb.domain, p, k);
    int X[3];
    if (!int_coords(pb.L, p, k, X)) break;
    if (first) {
      // first move out of the borrowed cell: copy its ancestors
      for (int l = 0; l < c.level; ++l) stk[l * stride] = sc->stk[l * stride];
    }
    first = false;
    relocate(pb, X, stk, stride, c);
  }
  return tau;
}

// Optical depth from p along k to the domain border at fixed x_ext (the
// peel-off integral); stops once tau >= tau_cut.  Uses its own LDS stack.
template <class R, int NL = MAX_LINES>
__device__ double ray_tau(const ProblemK &pb, const double p0[3], const double k[3], double x_ext,
                          double tau_cut, int *stk, int stride, uint32_t *ncross,
                          const StartCell<R> *sc, const double *kinv = nullptr) {
  double p[3] = {p0[0], p0[1], p0[2]};
  Cell c;
  const bool reuse = sc && strictly_inside(*sc->c, pb.L, p);
  if (reuse) {
    c = *sc->c;
  } else {
    int X[3];
    if (!int_coords(pb.L, p, k, X)) return 0.0;
    locate(pb, X, stk, stride, c);
  }
  return ray_walk<R, NL>(pb, p, k, x_ext, 0.0, 0u, tau_cut, stk, stride, ncross, c, sc, reuse, kinv);
}

// Pixel of position p in observer ob's image, -1 outside.  The double path
// bins exactly as the oracle does (divide by the span); the float path
// multiplies by the precomputed cells per unit (a point within an ulp of a
// pixel edge may fall on the other side).
template <bool FAST = false>
__device__ __forceinline__ int pixel_of(const ObsK &ob, const double p[3]) {
#pragma clang fp contract(off)
  const double q0 = p[0] - 0.5, q1 = p[1] - 0.5, q2 = p[2] - 0.5;
  const double u = q0 * ob.e1[0] + q1 * ob.e1[1] + q2 * ob.e1[2];
  const double v = q0 * ob.e2[0] + q1 * ob.e2[1] + q2 * ob.e2[2];
  const double fu = FAST ? (u - ob.u0) * ob.su : (u - ob.u0) / ob.uspan * ob.nx;
  const double fv = FAST ? (v - ob.v0) * ob.sv : (v - ob.v0) / ob.vspan * ob.ny;
  if (!(fu >= 0.0 && fu < ob.nx && fv >= 0.0 && fv < ob.ny)) return -1;
  const int ix = (int)floor(fu), iy = (int)floor(fv);
  if (ix >= ob.nx || iy >= ob.ny) return -1;
  return iy * ob.nx + ix;
}

template <bool FAST = false>
__device__ __forceinline__ int bin_of(const ObsK &ob, double x) {
#pragma clang fp contract(off)
  const double fb = FAST ? (x - ob.x_min) * ob.sx : (x - ob.x_min) / ob.xspan * ob.nbins;
  if (!(fb >= 0.0 && fb < ob.nbins)) return -1;
  const int b = (int)floor(fb);
  return b >= ob.nbins ? -1 : b;
}

struct LaneCount {
  uint32_t cross, peel_rays, peel_cross, peel_drop, dust_scat;
};

// What a scattering (or emission) needs to be redone toward an observer.
template <class R> struct PeelSrc {
  int kind;        // 0 emission, 1 line, 2 dust, 3 fluorescent re-emission
  R kin[3];
  R x;             // emission / dust: x_ext of the packet; line: cell-frame x
  R w;             // k_in . u of the cell (dust)
  R U[3];          // atom velocity / v_th of the line (line)
  R bc;            // v_th,line,cell / c (line)
  R rho;           // sqrt(T/T_ref) (line)
  R irho;          // 1/rho (line)
  int line, core;  // (fluorescent: core holds the channel)
  R ux, uy, uz;    // cell bulk velocity / v_th,ref
};

// Where a transport wave queues its deferred peel-off rays: its own region
// of the queue and the region's fill count, kept in LDS (one per wave, so
// no global atomics).  The wave stops taking events before the region
// could overflow, so a push always finds room.
template <class R> struct PeelSink {
  PeelJob<R> *region;
  int *count;
  uint32_t cap;
  unsigned long long *lost;   // pushes that found no room (never expected)
};

// First-leaf test of a peel-off ray toward observer ob from p, in the
// scattering's own leaf (its record is in the lane's registers; the leaf
// lies strictly inside the domain): true if the optical depth to the exit
// face along k_obs already reaches the cut, where exp(-tau) is zero and no
// deposit changes.  Without EXIT (float path) that distance alone is
// computed; with EXIT (double path, deferred rays) the nearest face is
// tried first, and a ray that goes on gets where it leaves the leaf (q,
// wrapped through periodic borders) and the optical depth so far.
template <class R, int NL, bool EXIT>
__device__ __forceinline__ bool peel_first_leaf(const ProblemK &pb, const double p[3], const ObsK &ob,
                                                const R ko[3], R xo, const StartCell<R> *sc, double q[3],
                                                double *qtau) {
  Opac<R, NL> o;
  opacity(pb, *sc->lf, (double)xo, ko, o);
  const double kt = (double)o.ktot;
  if constexpr (!EXIT) {
    // the distance to the leaf's face ahead along k_obs, as exit_dist
    // computes it (the observer's direction is uniform across the wave)
    const double inv = ldexp(1.0, -pb.L);
    const int sz = 1 << (pb.L - sc->c->level);
    const int o3[3] = {sc->c->ox, sc->c->oy, sc->c->oz};
    double te = __builtin_inf();
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      if (ob.k[d] != 0.0) {
        const double f = (double)(ob.k[d] > 0.0 ? o3[d] + sz : o3[d]) * inv;
        const double t = (f - p[d]) * ob.kinv[d];
        te = t < te ? t : te;
      }
    }
    return kt * (te < 0.0 ? 0.0 : te) >= TauCut<R>::v;
  }
  if (kt * inner_dist(*sc->c, pb.L, p) >= TauCut<R>::v) return true;
  double face[3], lo[3], hi[3];
  int em;
  const double te = exit_dist(*sc->c, pb.L, p, ob.k, face, lo, hi, &em, sizeof(R) == 4 ? ob.kinv : nullptr);
  const double t1 = kt * te;
  if (t1 >= TauCut<R>::v) return true;
  if constexpr (EXIT) {
    exit_point(te, em, p, ob.k, face, lo, hi, q);
    wrap_slab(pb.domain, q, ob.k);
    *qtau = t1;
  }
  return false;
}

// Queue a peel-off ray for the ray-cast pass, which makes every deposit:
// the float path queues it from its start (the pass walks the first leaf
// again, which keeps this kernel's registers low enough for four waves per
// SIMD), the double path, when its first leaf was tested, from where it
// leaves that leaf with the optical depth so far (qsteps = 1).  One LDS
// atomic per wave reserves the slots of the lanes pushing here.
template <class R>
__device__ __forceinline__ void peel_push(const ProblemK &pb, const double q[3], double qtau, uint32_t qsteps,
                                          R xo, R weight, size_t elem, int oi, const PeelSink<R> &snk) {
  const unsigned long long m = __ballot(true);
  const int lane = __lane_id();
  const int leader = __ffsll((long long)m) - 1;
  int base = 0;
  if (lane == leader) base = atomicAdd(snk.count, __popcll(m));
  base = __shfl(base, leader);
  const uint32_t slot = (uint32_t)base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
  if (slot < snk.cap) {
    PeelJob<R> &j = snk.region[slot];
    j.p[0] = q[0]; j.p[1] = q[1]; j.p[2] = q[2];
    j.x = xo;
    j.weight = weight;
    j.dst = (unsigned long long)elem | ((unsigned long long)oi << PQ_OBS_SHIFT) |
            ((unsigned long long)pb.index << PQ_PROB_SHIFT);
    if constexpr (sizeof(R) == 8) {
      j.tau = qtau;
      j.steps = qsteps;
    }
  } else {
    atomicAdd(snk.lost, 1ull);
  }
}

// Peel-off of one event toward every observer (Sect. 5.1).  A ray from a
// leaf strictly inside the domain is first tested in that leaf, before its
// weight, pixel and bin are computed: most rays from optically thick gas
// end there with no deposit.  A ray that goes on is binned (deposits
// outside the cube are dropped and counted) and, with DEFER, queued for the
// ray-cast pass (peel_push), else walked here; the float path queues it
// unbinned, and the pass bins it.  Emission rays (sc null: no
// leaf located yet) and rays from leaves the domain border may cut skip the
// first-leaf test.
template <class R, bool DEFER, int NL>
__device__ void peel_all(const ProblemK &pb, const double p[3], const PeelSrc<R> &s, int *stk,
                         int stride, LaneCount &cnt, const PeelSink<R> &snk, const StartCell<R> *sc = nullptr) {
  for (int oi = 0; oi < pb.n_obs; ++oi) {
    const ObsK &ob = pb.obs[oi];
    const R ko[3] = {cst<R>(ob.k[0], ob.kf[0]), cst<R>(ob.k[1], ob.kf[1]), cst<R>(ob.k[2], ob.kf[2])};
    R xo, mu = R(0);
    if (s.kind == 0) {
      xo = s.x;
    } else if (NL > 1 && s.kind == 3) {
      // fluorescent re-emission: isotropic, at the channel's rest frequency
      // in the atom frame, then through the cell's velocity
      const LineK &ln = pb.lines[s.line];
      const R ba = s.bc * (ko[0] * s.U[0] + ko[1] * s.U[1] + ko[2] * s.U[2]);
      const R bw = cst<R>(pb.b_ref, pb.b_ref_f) * (ko[0] * s.ux + ko[1] * s.uy + ko[2] * s.uz);
      xo = cst<R>(ln.xf0[s.core], ln.f.xf0[s.core]) + M<R>::div(cst<R>(ln.sf[s.core], ln.f.sf[s.core]) * (ba + bw + ba * bw), cst<R>(pb.b_ref, pb.b_ref_f));
    } else if (s.kind == 1) {
      const LineK &ln = pb.lines[s.line];
      mu = s.kin[0] * ko[0] + s.kin[1] * ko[1] + s.kin[2] * ko[2];
      const R dkU = (ko[0] - s.kin[0]) * s.U[0] + (ko[1] - s.kin[1]) * s.U[1] + (ko[2] - s.kin[2]) * s.U[2];
      const R g1 = R(1) + s.bc * s.x;
      const R Rr = ln.recoil ? (R(1) - mu) * cst<R>(ln.rec, ln.f.rec) * g1 : R(0);
      R xc;
      if constexpr (sizeof(R) == 4) {
        // Rr < 3e-8 for any line and scatterer (h nu <= 13.6 eV, m c^2 >=
        // 938 MeV): 1/(1 + Rr) = 1 - Rr to float precision, and
        // Rr/bc = Rr irho / (b_ref mu)
        xc = (s.x + g1 * dkU - Rr * cst<R>(ln.ibmu, ln.f.ibmu) * s.irho) * (R(1) - Rr);
      } else {
        xc = M<R>::div(s.x + g1 * dkU - M<R>::div(Rr, s.bc), R(1) + Rr);
      }
      const R wo = ko[0] * s.ux + ko[1] * s.uy + ko[2] * s.uz;
      xo = (-cst<R>(ln.delta, ln.f.delta) + cst<R>(ln.mu, ln.f.mu) * s.rho * xc * (R(1) + cst<R>(pb.b_ref, pb.b_ref_f) * wo) + wo) * cst<R>(ln.inv_s, ln.f.inv_s);
    } else {
      mu = s.kin[0] * ko[0] + s.kin[1] * ko[1] + s.kin[2] * ko[2];
      const R wo = ko[0] * s.ux + ko[1] * s.uy + ko[2] * s.uz;
      const R b = cst<R>(pb.b_ref, pb.b_ref_f);
      xo = M<R>::div(s.x + wo + b * s.x * wo - s.w, R(1) + b * s.w);
    }
    ++cnt.peel_rays;
    constexpr bool EXIT = DEFER && sizeof(R) == 8;
    double q[3] = {p[0], p[1], p[2]}, qtau = 0.0;
    uint32_t qsteps = 0;
    if (sc && sc->lf->bnd == R(0)) {
      if (peel_first_leaf<R, NL, EXIT>(pb, p, ob, ko, xo, sc, q, &qtau)) {
        ++cnt.peel_cross;
        continue;
      }
      qsteps = EXIT ? 1u : 0u;
    }
    R weight;
    if (s.kind == 0 || (NL > 1 && s.kind == 3)) {
      weight = R(1.0 / (4.0 * PI_D));
    } else if (s.kind == 1) {
      const LineK &ln = pb.lines[s.line];
      const R P = ln.phase == PHASE_ISO ? R(0.5) : (s.core ? p_core(mu) : p_wing(mu));
      weight = P * R(1.0 / (2.0 * PI_D));
    } else {
      weight = p_hg(mu, cst<R>(pb.g_hg, pb.g_hg_f)) * R(1.0 / (2.0 * PI_D));
    }
    if constexpr (DEFER && sizeof(R) == 4) {
      // the float ray-cast pass bins the ray from its start (and counts
      // the deposits outside the cube)
      peel_push<R>(pb, q, 0.0, 0u, xo, weight, 0, oi, snk);
      continue;
    }
    const int pix = pixel_of<sizeof(R) == 4>(ob, p);
    const int bin = bin_of<sizeof(R) == 4>(ob, (double)xo);
    if (pix < 0 || bin < 0) {
      ++cnt.peel_drop;
      continue;
    }
    const size_t elem = (size_t)pix * ob.nbins + bin;
    if constexpr (DEFER) {
      if (qsteps) ++cnt.peel_cross;
      peel_push<R>(pb, q, qtau, qsteps, xo, weight, elem, oi, snk);
    } else {
      uint32_t nc = 0;
      const double tau = ray_tau<R, NL>(pb, p, ob.k, (double)xo, TauCut<R>::v, stk, stride, &nc, sc,
                                        sizeof(R) == 4 ? ob.kinv : nullptr);
      cnt.peel_cross += nc;
      if (tau < TauCut<R>::v) atomic_add_real((R *)ob.cube + elem, weight * M<R>::exp((R)(-tau)));
    }
  }
}

// ------------------------------------------------------------- transport
template <class R> struct Lane {
  int64_t pid;
  double p[3];
  R k[3];
  double kd[3];    // direction used for geometry (unit in double)
  R x;
  double tau, path;
  uint32_t event;
  uint32_t rej;    // regrouped loop: rejection rounds already run by the pending
                   // line scattering at p (0: none pending)
  int32_t nscat;
  Cell c;
  LeafRec<R> lf;
  LaneCount cnt;
};

// Geometry direction: the float direction of the bulk path is renormalised
// in double so that a packet's displacement equals its path length.
template <class R> __device__ __forceinline__ void set_geom_dir(Lane<R> &s) {
  if constexpr (sizeof(R) == 4) {
    const double a = s.k[0], b = s.k[1], c = s.k[2];
    // |k|^2 = 1 + e with |e| of order the float rounding: 1/sqrt(1+e) by its
    // series to e^3 (remainder below 2^-53 for |e| < 2^-16), else exactly
    const double e = fma(a, a, fma(b, b, fma(c, c, -1.0)));
    const double inv = fabs(e) < 0x1p-16 ? 1.0 + e * (-0.5 + e * (0.375 - 0.3125 * e)) : 1.0 / sqrt(1.0 + e);
    s.kd[0] = a * inv; s.kd[1] = b * inv; s.kd[2] = c * inv;
  } else {
    s.kd[0] = s.k[0]; s.kd[1] = s.k[1]; s.kd[2] = s.k[2];
  }
}

// Record a packet that ended (escaped, absorbed or stuck): its outputs and
// its counts.  Ends are counted in the wave's LDS counters ends[status - 1]
// and published once per launch: with an atomic on the run's counters per
// wave and loop pass, packets with short walks queued on those few addresses
// (the Fe II wind, 2e6 packets: four such atomics and one on the queue per
// group of ends took most of 24.7 ms; 3.8 ms without them).  Single-problem launches publish the packets' work (scatterings,
// crossings, peel-off rays) with the launch's slice totals at the end of the
// kernel; in batches, whose lanes change problem, each packet adds its own
// to its problem's totals here.  Dropped peel-off deposits are reported in
// the slice where their packet ends.
template <class R, bool BATCH>
__device__ void finish(const ProblemK &pb, Lane<R> &s, int status, int *ends, unsigned long long *slice) {
  const int64_t i = s.pid - pb.first;
  pb.status[i] = status;
  pb.x_out[i] = (double)s.x;
  pb.k_out[3 * i] = (double)s.k[0];
  pb.k_out[3 * i + 1] = (double)s.k[1];
  pb.k_out[3 * i + 2] = (double)s.k[2];
  pb.pos_out[3 * i] = s.p[0];
  pb.pos_out[3 * i + 1] = s.p[1];
  pb.pos_out[3 * i + 2] = s.p[2];
  pb.nscat[i] = s.nscat;
  pb.path_out[i] = s.path;
  unsigned long long *st = pb.stats;
  atomicAdd(ends + (status - 1), 1);
  if (BATCH) {
    atomicAdd(st + S_EMITTED, 1ull);
    atomicAdd(st + S_ESCAPED + (status - 1), 1ull);
    atomicAdd(st + S_SCAT, (unsigned long long)s.nscat);
    if (s.cnt.dust_scat) atomicAdd(st + S_DUST_SCAT, (unsigned long long)s.cnt.dust_scat);
    atomicAdd(st + S_CROSS, (unsigned long long)s.cnt.cross);
    if (s.cnt.peel_rays) atomicAdd(st + S_PEEL_RAYS, (unsigned long long)s.cnt.peel_rays);
    if (s.cnt.peel_cross) atomicAdd(st + S_PEEL_CROSS, (unsigned long long)s.cnt.peel_cross);
  }
  if (s.cnt.peel_drop) {
    atomicAdd(st + S_PEEL_DROPPED, (unsigned long long)s.cnt.peel_drop);
    atomicAdd(slice + S_PEEL_DROPPED, (unsigned long long)s.cnt.peel_drop);
  }
}

// Emission (Sect. 2): position and frequency from the source list,
// isotropic direction unless given, tau_event = -ln r.
// Source spectrum (Sect. 2.1), added to the source's own x, in double in
// both precisions, by a pass before the transport (k_source_x) so that the
// transport kernels carry none of it.  Gaussian line: Box-Muller draw times
// sigma (Doppler widths of the reference line).  Power-law continuum,
// F_lambda ~ lambda^beta on [lambda_min, lambda_max]: inverse CDF of the
// photon-number distribution lambda F_lambda, then
// x = (lambda_ref - lambda) / (lambda b_ref)  (nu = c / lambda).
// r1, r2: the packet's emission draws J_SRC1, J_SRC2.
__device__ inline double source_spectrum_x(const ProblemK &pb, double r1, double r2) {
  if (pb.spec_kind == 1) return pb.spec_p[0] * sqrt(-2.0 * log(r1)) * cospi(2.0 * r2);
  if (pb.spec_kind == 3) {
    // tabulated continuum: bin i with probability (cum[i+1] - cum[i]) / cum[n-1]
    // (bisection), then the bin's power law by its inverse CDF in ratio form
    const double t = r1 * pb.tab_cum[pb.tab_n - 1];
    int lo = 0, hi = pb.tab_n - 2;  // the bin: first i with t < cum[i+1]
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (t < pb.tab_cum[mid + 1]) hi = mid; else lo = mid + 1;
    }
    const double l0 = pb.tab_lam[lo], l1 = pb.tab_lam[lo + 1], b = pb.tab_beta[lo];
    double lam;
    if (b == -2.0) {
      lam = l0 * exp(r2 * log(l1 / l0));
    } else {
      const double e = 2.0 + b;
      lam = l0 * pow(1.0 + r2 * (pow(l1 / l0, e) - 1.0), 1.0 / e);
    }
    return (pb.lambda_ref - lam) / (lam * pb.b_ref);
  }
  const double lmin = pb.spec_p[0], lmax = pb.spec_p[1], beta = pb.spec_p[2];
  const double r = r1;
  double lam;
  if (beta == -2.0) {
    lam = lmin * exp(r * log(lmax / lmin));
  } else {
    const double e = 2.0 + beta, a = pow(lmin, e);
    lam = pow(a + r * (pow(lmax, e) - a), 1.0 / e);
  }
  return (pb.lambda_ref - lam) / (lam * pb.b_ref);
}

// x_out[pid] = src_x[pid] + the packet's spectral draw, for pid in
// [first, first + n): the same counter-based emission draws (event 0,
// slots J_SRC1 and J_SRC2) the transport's precision would take.
template <class R>
__global__ void __launch_bounds__(256) k_source_x(const ProblemK pb, const double *__restrict__ src_x,
                                                  double *__restrict__ x_out, int64_t first, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t pid = first + i;
  EventRng<R> rng(pb.seed, (uint64_t)pid, 0u);
  const double r1 = (double)rng.u(J_SRC1), r2 = (double)rng.u(J_SRC2);
  x_out[pid] = src_x[pid] + source_spectrum_x(pb, r1, r2);
}

hipError_t launch_source_x(bool f32, const ProblemK &pb, const double *src_x, double *x_out, int64_t first,
                           int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (f32)
    hipLaunchKernelGGL(k_source_x<float>, dim3(blocks), dim3(256), 0, stream, pb, src_x, x_out, first, n);
  else
    hipLaunchKernelGGL(k_source_x<double>, dim3(blocks), dim3(256), 0, stream, pb, src_x, x_out, first, n);
  return hipGetLastError();
}

template <class R, bool DEFER, int NL>
__device__ void emit(const ProblemK &pb, int64_t pid, Lane<R> &s, int *stk, int *pstk, int stride,
                     const PeelSink<R> &snk) {
  s.pid = pid;
  s.p[0] = pb.src_pos[3 * pid];
  s.p[1] = pb.src_pos[3 * pid + 1];
  s.p[2] = pb.src_pos[3 * pid + 2];
  EventRng<R> rng(pb.seed, (uint64_t)pid, 0u);
  if (pb.src_dir) {
    s.k[0] = (R)pb.src_dir[3 * pid];
    s.k[1] = (R)pb.src_dir[3 * pid + 1];
    s.k[2] = (R)pb.src_dir[3 * pid + 2];
  } else {
    const R mu = R(2) * rng.u(J_MU) - R(1);
    R sp, cp;
    M<R>::sincos2pi(rng.u(J_PHI), &sp, &cp);
    const R st = M<R>::sqrt(R(1) - mu * mu);
    s.k[0] = st * cp;
    s.k[1] = st * sp;
    s.k[2] = mu;
  }
  set_geom_dir(s);
  s.x = (R)pb.src_x[pid];
  s.tau = -(double)M<R>::log(rng.u(J_TAU));
  s.path = 0.0;
  s.event = 0;
  s.nscat = 0;
  s.rej = 0;
  s.cnt = LaneCount{0, 0, 0, 0, 0};
  if (pb.n_obs) {
    PeelSrc<R> ps;
    ps.kind = 0;
    ps.x = s.x;
    peel_all<R, DEFER, NL>(pb, s.p, ps, pstk, stride, s.cnt, snk);
  }
}

// Sums of products with the fused ones named, so that every kernel that
// inlines them rounds alike (the walkers' kernel gets the sines and cosines
// from elsewhere than the bulk kernels, and the compiler would pick other
// products to fuse).
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }
// a b + c d with c d rounded first
template <class R> __device__ __forceinline__ R dot2(R a, R b, R c, R d) {
  const R t = c * d;
  return fmadd(a, b, t);
}
// (a0 b0 + a1 b1) + a2 b2 with a1 b1 rounded first
template <class R> __device__ __forceinline__ R dot3(R a0, R b0, R a1, R b1, R a2, R b2) {
  return fmadd(a2, b2, dot2(a0, b0, a1, b1));
}
// The direction at angle cosine mu (sine st) from kin and azimuth (sp, cp)
// in the plane of e1, e2.
template <class R>
__device__ __forceinline__ void rotate(R k[3], R mu, R st, R sp, R cp, const R kin[3], const R e1[3], const R e2[3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const R t = sizeof(R) == 4 ? dot2(cp, e1[d], sp, e2[d]) : dot2(sp, e2[d], cp, e1[d]);
    k[d] = dot2(mu, kin[d], st, t);
  }
}

// The draws of one event in the order the interaction takes them, computed
// where they are used (bulk kernels).
template <class R, bool REGROUP> struct RngDraws {
  EventRng<R> rng;
  R r_late, r_mu, r_p1, r_p2, r_phi;
  __device__ __forceinline__ RngDraws(const ProblemK &pb, const Lane<R> &s) : rng(pb.seed, (uint64_t)s.pid, s.event) {}
  // kappa_d / kappa reaches ~1e-8 in optically thick line cores
  __device__ __forceinline__ R channel() {
    const R r = rng.u_small(J_CHANNEL);
    // the double generator keeps one Philox block: the draw of the channel's
    // block that the event uses last (the scattering angle) is taken now, so
    // that no block of the event is computed twice; the float path takes the
    // draws of block 0 it needs late now (tau_event and the scattering angle),
    // which leaves that block's words dead after the first rejection round
    r_late = rng.u(sizeof(R) == 4 ? J_TAU : J_MU);
    if constexpr (sizeof(R) == 4) r_mu = rng.u(J_MU);
    return r;
  }
  __device__ __forceinline__ R albedo() { return rng.u(J_ALBEDO); }
  __device__ __forceinline__ R mu() { return sizeof(R) == 8 ? r_late : r_mu; }
  __device__ __forceinline__ R log_tau() { return M<R>::log(sizeof(R) == 4 ? r_late : rng.u(J_TAU)); }
  // float: block 1 (the second rejection round, the perpendicular
  // velocities and the azimuth) for every lane of the line branch at once, its
  // outgoing draws taken now so that its words are dead after the
  // sampler's second round
  __device__ __forceinline__ void line() {
    if constexpr (sizeof(R) == 4) {
      rng.need1();
      r_p1 = rng.u(J_PERP1);
      r_p2 = rng.u(J_PERP2);
      r_phi = rng.u(J_PHI);
    }
  }
  __device__ __forceinline__ R log_perp() { return M<R>::log(sizeof(R) == 4 ? r_p1 : rng.u(J_PERP1)); }
  __device__ __forceinline__ void perp(R *sp, R *cp) { M<R>::sincos2pi(sizeof(R) == 4 ? r_p2 : rng.u(J_PERP2), sp, cp); }
  __device__ __forceinline__ void phi(R *sp, R *cp) { M<R>::sincos2pi(sizeof(R) == 4 ? r_phi : rng.u(J_PHI), sp, cp); }
  // (the dust branch has not taken block 1)
  __device__ __forceinline__ void phi_dust(R *sp, R *cp) { M<R>::sincos2pi(rng.u(J_PHI), sp, cp); }
  __device__ __forceinline__ R decay() { return rng.u(J_DECAY); }
  __device__ __forceinline__ R dipole(bool core) { return mu_dipole(mu(), core); }
  // The parallel atom velocity: false when the rounds run out, or (regrouped
  // draw) when this call's round is rejected; then undrawn() is the packet's
  // status (a pending event's packet lives on, with s.rej rounds run).
  __device__ __forceinline__ bool upar(Lane<R> &s, R x, R a, R la, R *out) {
    if constexpr (REGROUP) {
      if (!upar_round<R>(x, a, la, rng, s.rej, out)) return false;
      s.rej = 0;
      return true;
    } else {
      return sample_upar<R>(x, a, la, rng, out);
    }
  }
  static __device__ __forceinline__ int undrawn(Lane<R> &s) {
    return REGROUP && ++s.rej < MAX_REJECT ? ST_NONE : ST_STUCK;
  }
};

// Interaction at the current position (Sect. 3.2).  Returns the packet's
// status (ST_NONE while it lives).  dr gives the event's draws, peel(ps)
// takes what its peel-off needs.
// With REGROUP a line scattering runs one rejection round of its u_par
// draw per call: a rejected round leaves the event pending (s.rej rounds
// run) and the packet where it is, and the next pass of the transport loop
// calls again for the next round (the same draws as the looping sampler).
template <class R, int NL, class PB, class D, class P>
__device__ __forceinline__ int interact(const PB &pb, Lane<R> &s, const Opac<R, NL> &o, D &dr, P &&peel) {
  R r = dr.channel() * o.ktot;
  const R kin[3] = {s.k[0], s.k[1], s.k[2]};
  // the pair perpendicular to k_in is formed where it is used (after the
  // atom-velocity draw on the line branch, whose register peak it would
  // otherwise raise)
  R e1[3], e2[3];
  PeelSrc<R> ps;
  ps.kin[0] = kin[0]; ps.kin[1] = kin[1]; ps.kin[2] = kin[2];
  ps.ux = s.lf.ux; ps.uy = s.lf.uy; ps.uz = s.lf.uz;
  ps.w = o.w;
  if (r < o.kd) {
    // dust (Sect. 3.2.2): absorbed with probability 1 - albedo, else HG
    if (dr.albedo() >= cst<R>(pb.albedo, pb.albedo_f)) return ST_ABSORBED;
    ++s.cnt.dust_scat;
    if (pb.n_obs) {
      ps.kind = 2;
      ps.x = s.x;
      peel(ps);
    }
    if (!pb.forward_only) {
      perp_basis(kin, e1, e2);
      const R mu = mu_hg(dr.mu(), cst<R>(pb.g_hg, pb.g_hg_f));
      R sp, cp;
      dr.phi_dust(&sp, &cp);
      const R st = M<R>::sqrt(fmax(R(0), R(1) - mu * mu));
      rotate(s.k, mu, st, sp, cp, kin, e1, e2);
      set_geom_dir(s);
      // coherent in the cell frame
      const R wn = s.k[0] * s.lf.ux + s.k[1] * s.lf.uy + s.k[2] * s.lf.uz;
      const R b = cst<R>(pb.b_ref, pb.b_ref_f);
      s.x = M<R>::div(s.x + wn + b * s.x * wn - o.w, R(1) + b * o.w);
    }
  } else {
    // resonant scattering in line i (Sect. 3.2.1)
    r -= o.kd;
    // first line whose cumulative opacity exceeds r (the last line takes
    // any rounding remainder)
    int i = 0;
    R x = o.x[0];
    bool found = false;
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      if (!found && q < pb.n_lines) {
        if (r < o.kl[q] || q == pb.n_lines - 1) {
          i = q;
          x = o.x[q];
          found = true;
        } else {
          r -= o.kl[q];
        }
      }
    }
    const LineK &ln = line_of(pb, i);
    const R a = cst<R>(ln.alpha, ln.f.alpha) * s.lf.irho;
    // log10 a for the envelope: the double path adds the line's log10 alpha
    // and the leaf's log10(1/rho) (its record holds it)
    const R la = sizeof(R) == 8 ? R(ln.lalpha) + s.lf.lg : M<R>::log10(a);
    dr.line();
    R upar;
    if (!dr.upar(s, x, a, la, &upar)) return dr.undrawn(s);
    // Gaussian u_perp (Box-Muller), restricted to |u_perp| >= x_crit while
    // core-skipping applies
    const R xc2 = pb.skip_tau > 0.0 ? core_skip_x2<R>(pb, ln, s.lf, s.c.level, a, x) : R(0);
    perp_basis(kin, e1, e2);
    R sp, cp;
    dr.perp(&sp, &cp);
    const R rr = M<R>::sqrt(xc2 - dr.log_perp());
    const R up1 = rr * cp, up2 = rr * sp;
    R U[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) U[d] = fmadd(up2, e2[d], dot2(upar, kin[d], up1, e1[d]));
    const R rho = M<R>::div(R(1), s.lf.irho);
    const R bc = cst<R>(pb.b_ref, pb.b_ref_f) * cst<R>(ln.mu, ln.f.mu) * rho;
    // frequency seen by the atom, nu_in (1 - k_in.v/c), within 0.2 dnu_D
    const R g1 = R(1) + bc * x;
    const int core = fabs(x - g1 * upar) < R(0.2);
    // decay channel (Sect. 3.2.1): fluorescent channel j when the draw lies
    // at or above A_ul / sum A (then (A_ul + A_0) / sum A for j = 1); lines
    // with channels run in the multi-line kernels only
    int fch = -1;
    if constexpr (NL > 1) {
      if (ln.n_fluor > 0 && !pb.forward_only) {
        const R ud = dr.decay();
        if (ud >= cst<R>(ln.a_res, ln.f.a_res)) fch = (ln.n_fluor > 1 && ud >= cst<R>(ln.a_cum0, ln.f.a_cum0)) ? 1 : 0;
      }
    }
    ++s.nscat;
    if (NL > 1 && fch >= 0) {
      if (pb.n_obs) {
        ps.kind = 3;
        ps.U[0] = U[0]; ps.U[1] = U[1]; ps.U[2] = U[2];
        ps.bc = bc;
        ps.line = i;
        ps.core = fch;
        peel(ps);
      }
      const R mu = R(2) * dr.mu() - R(1);
      dr.phi(&sp, &cp);
      const R st = M<R>::sqrt(fmax(R(0), R(1) - mu * mu));
      rotate(s.k, mu, st, sp, cp, kin, e1, e2);
      set_geom_dir(s);
      const R ku = dot3(s.k[0], U[0], s.k[1], U[1], s.k[2], U[2]);
      const R bw = cst<R>(pb.b_ref, pb.b_ref_f) * dot3(s.k[0], s.lf.ux, s.k[1], s.lf.uy, s.k[2], s.lf.uz);
      const R ba = bc * ku;
      const R shift = fmadd(ba, bw, fmadd(bc, ku, bw));   // ba + bw + ba bw
      s.x = cst<R>(ln.xf0[fch], ln.f.xf0[fch]) + M<R>::div(cst<R>(ln.sf[fch], ln.f.sf[fch]) * shift, cst<R>(pb.b_ref, pb.b_ref_f));
      s.tau = -(double)dr.log_tau();
      return ST_NONE;
    }
    if (pb.n_obs) {
      ps.kind = 1;
      ps.x = x;
      ps.U[0] = U[0]; ps.U[1] = U[1]; ps.U[2] = U[2];
      ps.bc = bc;
      ps.rho = rho;
      ps.irho = s.lf.irho;
      ps.line = i;
      ps.core = core;
      peel(ps);
    }
    if (!pb.forward_only) {
      const R mu = ln.phase == PHASE_ISO ? R(2) * dr.mu() - R(1) : dr.dipole(core != 0);
      dr.phi(&sp, &cp);
      const R st = M<R>::sqrt(fmax(R(0), R(1) - mu * mu));
      rotate(s.k, mu, st, sp, cp, kin, e1, e2);
      set_geom_dir(s);
      // outgoing frequency, coherent in the atom frame, recoil in the
      // denominator (Eq. for nu_out), then back to the external frame
      const R dkU = dot3(s.k[0] - kin[0], U[0], s.k[1] - kin[1], U[1], s.k[2] - kin[2], U[2]);
      const R Rr = ln.recoil ? (R(1) - mu) * cst<R>(ln.rec, ln.f.rec) * g1 : R(0);
      R xc;
      if constexpr (sizeof(R) == 4) {
        // as in the peel-off: 1/(1 + Rr) = 1 - Rr and Rr/bc = Rr irho/(b_ref mu)
        xc = (x + g1 * dkU - Rr * cst<R>(ln.ibmu, ln.f.ibmu) * s.lf.irho) * (R(1) - Rr);
      } else {
        xc = M<R>::div(x + g1 * dkU - M<R>::div(Rr, bc), R(1) + Rr);
      }
      const R wn = s.k[0] * s.lf.ux + s.k[1] * s.lf.uy + s.k[2] * s.lf.uz;
      s.x = (-cst<R>(ln.delta, ln.f.delta) + cst<R>(ln.mu, ln.f.mu) * rho * xc * (R(1) + cst<R>(pb.b_ref, pb.b_ref_f) * wn) + wn) * cst<R>(ln.inv_s, ln.f.inv_s);
    }
  }
  s.tau = -(double)dr.log_tau();
  return ST_NONE;
}

// Packet state kept in HBM between launches (one slot per lane of the
// grid): a run is a sequence of bounded launches, each lane resuming the
// packet it held, so no launch waits for the longest random walk and each
// launch can be replayed from a captured graph.
struct SlotState {
  double p[3], k[3];
  double x, tau, path;
  int64_t pid;
  int32_t prob, active, event, nscat;
  int32_t leaf, level, ox, oy, oz;
  uint32_t dust, cross, peel_rays, peel_cross, peel_drop;
  uint32_t rej;
};

template <class R>
__device__ __forceinline__ void save_slot(SlotState &q, const Lane<R> &s, int prob) {
  for (int d = 0; d < 3; ++d) { q.p[d] = s.p[d]; q.k[d] = (double)s.k[d]; }
  q.x = (double)s.x; q.tau = s.tau; q.path = s.path; q.pid = s.pid;
  q.prob = prob; q.active = 1; q.event = (int32_t)s.event; q.nscat = s.nscat;
  q.leaf = s.c.leaf; q.level = s.c.level; q.ox = s.c.ox; q.oy = s.c.oy; q.oz = s.c.oz;
  q.dust = s.cnt.dust_scat; q.cross = s.cnt.cross; q.peel_rays = s.cnt.peel_rays;
  q.peel_cross = s.cnt.peel_cross; q.peel_drop = s.cnt.peel_drop;
  q.rej = s.rej;
}

template <class R>
__device__ __forceinline__ void load_slot(const SlotState &q, Lane<R> &s, int *prob) {
  for (int d = 0; d < 3; ++d) { s.p[d] = q.p[d]; s.k[d] = (R)q.k[d]; }
  s.x = (R)q.x; s.tau = q.tau; s.path = q.path; s.pid = q.pid;
  *prob = q.prob; s.event = (uint32_t)q.event; s.nscat = q.nscat;
  s.c.leaf = q.leaf; s.c.level = q.level; s.c.ox = q.ox; s.c.oy = q.oy; s.c.oz = q.oz;
  s.cnt.dust_scat = q.dust; s.cnt.cross = q.cross; s.cnt.peel_rays = q.peel_rays;
  s.cnt.peel_cross = q.peel_cross; s.cnt.peel_drop = q.peel_drop;
  s.rej = q.rej;
  set_geom_dir(s);
}

// Counters of work done inside one launch, summed over the wave and
// published at the kernel's end (the packets that end in it are counted by
// finish).
struct SliceCount {
  uint32_t scat, dust, cross, peel_rays, peel_cross;
};

template <class R>
__device__ __forceinline__ void add_delta(SliceCount &a, const Lane<R> &s, const Lane<R> &z) {
  a.scat += (uint32_t)(s.nscat - z.nscat);
  a.dust += s.cnt.dust_scat - z.cnt.dust_scat;
  a.cross += s.cnt.cross - z.cnt.cross;
  a.peel_rays += s.cnt.peel_rays - z.cnt.peel_rays;
  a.peel_cross += s.cnt.peel_cross - z.cnt.peel_cross;
}

// A wave's counts of one launch into the launch's slice counters and, unless
// null, a problem's totals: its lanes' work and the packets that ended
// (ends[status - 1]).  Every lane calls it.
__device__ __forceinline__ void publish(unsigned long long *stats, const SliceCount &acc, const int *ends,
                                        unsigned long long *slice) {
  const int lane = __lane_id();
  if (lane == 0) {
    unsigned long long n = 0;
    for (int j = 0; j < 3; ++j) {
      const unsigned long long e = (unsigned long long)(uint32_t)ends[j];
      n += e;
      if (e) {
        atomicAdd(slice + S_ESCAPED + j, e);
        if (stats) atomicAdd(stats + S_ESCAPED + j, e);
      }
    }
    if (n) {
      atomicAdd(slice + S_EMITTED, n);
      if (stats) atomicAdd(stats + S_EMITTED, n);
    }
  }
  const unsigned long long v[5] = {acc.scat, acc.dust, acc.cross, acc.peel_rays, acc.peel_cross};
  const int idx[5] = {S_SCAT, S_DUST_SCAT, S_CROSS, S_PEEL_RAYS, S_PEEL_CROSS};
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    unsigned long long x = v[j];
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off);
    if (lane == 0 && x) {
      atomicAdd(slice + idx[j], x);
      if (stats) atomicAdd(stats + idx[j], x);
    }
  }
}

// The first active lane's value, as a wave-uniform one.
__device__ __forceinline__ unsigned long long uniform64(unsigned long long v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (unsigned long long)hi << 32 | lo;
}

// Idle lane passes a wave gathers before it records its ended packets and
// takes new ones.  A refill (emission, point location, the ended packets'
// outputs) costs the wave about as many instructions as one loop pass does
// for its 64 lanes whether one lane or all take part, so waiting until 64
// lane passes were idle at most doubles the smaller of the two costs (the
// Fe II wind, 2e6 packets of 48 crossings: 5.6 ms without the wait, 3.9 at
// 24, 3.8 at 64 and 128; long walks: no difference).
#ifndef RMC_REFILL_DEBT
#define RMC_REFILL_DEBT 64
#endif
constexpr uint32_t REFILL_DEBT = RMC_REFILL_DEBT;

// A transport wave's words in LDS: peel-off rays queued, packets that escaped,
// were absorbed, got stuck; passes run when the queue was last found dry; packets
// started; whether the queue is long; the wave's reserve [next, end) of it, 64
// bits each.
enum { WAVE_QUEUED = 0, WAVE_ENDS = 1, WAVE_DRY = 4, WAVE_STARTED, WAVE_PLENTY, WAVE_NEXT = 8, WAVE_END = 10, WAVE_WORDS = 12 };
__device__ __forceinline__ void put64(int *p, unsigned long long v) {
  p[0] = (int)(uint32_t)v;
  p[1] = (int)(uint32_t)(v >> 32);
}
__device__ __forceinline__ unsigned long long get64(const int *p) {
  return uniform64((unsigned long long)(uint32_t)p[1] << 32 | (uint32_t)p[0]);
}

// Waves per SIMD the transport kernel is compiled for (register budget,
// chosen by measurement): the float single-problem kernels with deferred
// peel-off run four (5 registers spill with one line, 7 with two, 14 with
// four, and they are 8-9% faster than at three), the other float kernels three
// (no spills with deferred peel-off; at four the batch kernels spill 50-90
// registers and the batch runs slower), the single-problem double kernels with
// deferred peel-off two (33-44 registers spill, and the dusty sphere runs 38%
// faster than at one, where nothing spills), the other double kernels (batch,
// inline walker; 90-200 registers would spill at two) one.
#ifndef RMC_WAVES_F32_LEAN
#define RMC_WAVES_F32_LEAN 4
#endif
#ifndef RMC_WAVES_F32
#define RMC_WAVES_F32 3
#endif
#ifndef RMC_WAVES_F32_MULTI
#define RMC_WAVES_F32_MULTI 4
#endif
#ifndef RMC_WAVES_F64
#define RMC_WAVES_F64 2
#endif
#ifndef RMC_WAVES_F64_WIDE
#define RMC_WAVES_F64_WIDE 1
#endif
template <class R, bool BATCH, bool DEFER, int NL> struct WavesPerEU;
template <bool BATCH, bool DEFER, int NL> struct WavesPerEU<float, BATCH, DEFER, NL> {
  static constexpr int v = (!BATCH && DEFER) ? (NL == 1 ? RMC_WAVES_F32_LEAN : RMC_WAVES_F32_MULTI) : RMC_WAVES_F32;
};
template <bool BATCH, bool DEFER, int NL> struct WavesPerEU<double, BATCH, DEFER, NL> {
  static constexpr int v = (!BATCH && DEFER) ? RMC_WAVES_F64 : RMC_WAVES_F64_WIDE;
};

constexpr int DRY_CHECK = 256;   // loop iterations between two looks at the queue

// Whether every packet has been taken from the queue (other waves' atomics move it).
__device__ __forceinline__ bool queue_dry(const unsigned long long *next, int64_t total) {
  return uniform64(__hip_atomic_load(next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >= (unsigned long long)total;
}

// REGROUP: a line scattering whose rejection round fails stays pending and
// takes its next round at the next pass of the loop, where it runs in step
// with the other lanes' events (upar_round), instead of the wave looping
// until its last lane accepts.
template <class R, bool BATCH, bool DEFER, int NL, bool REGROUP = false>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(WavesPerEU<R, BATCH, DEFER, NL>::v, WavesPerEU<R, BATCH, DEFER, NL>::v)))
    k_transport(const ProblemK *__restrict__ probs,
                                                   const int64_t *__restrict__ starts, int n_probs,
                                                   unsigned long long *__restrict__ next,
                                                   int refill_min, int stack_levels,
                                                   SlotState *__restrict__ slots, int budget,
                                                   unsigned long long *__restrict__ slice) {
  extern __shared__ int lds[];
  const int stride = blockDim.x;
  int *stk = lds + threadIdx.x;
  int *pstk = lds + stack_levels * stride + threadIdx.x;
  const int64_t total = starts[n_probs];
  const int lane = __lane_id();
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // this wave's region of the deferred peel-off queue; the wave ends its
  // slice early once one more iteration (an emission and an event, each
  // peeled toward every observer) could overflow it
  // (no queue when no problem of the launch has an observer)
  PeelQueue *const pq = DEFER ? probs[0].pq : nullptr;
  const bool queue = DEFER && pq != nullptr;
  // (wave-uniform, and told so: what follows from it then stays in scalar registers)
  const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t wave = (int64_t)blockIdx.x * (stride >> 6) + wib;
  PeelSink<R> snk;
  // What the wave needs seldom, in LDS (WAVE_* words; every lane writes the same):
  // as values of the loop they took scalar registers whose spills cost vector ones
  // (dusty sphere without observer, launches of 8192 passes: FP64 66.8 -> 65.1 ms,
  // FP32 41.3 -> 39.5), and a value that left the loop by each of its exits would
  // cost the float kernels 150 spills.
  int *const wcnt = lds + 2 * stack_levels * stride + WAVE_WORDS * wib;
  snk.count = wcnt + WAVE_QUEUED;
  snk.region = queue ? (PeelJob<R> *)pq->jobs + (size_t)wave * pq->cap : nullptr;
  snk.cap = queue ? (uint32_t)pq->cap : 0u;
  snk.lost = queue ? &pq->lost : nullptr;
  const int room = queue ? (int)pq->cap - 2 * 64 * MAX_OBS : 0x7fffffff;
  if (lane < WAVE_WORDS) wcnt[lane] = 0;

  // the wave's reserve of packets taken from the queue and not started yet
  unsigned long long *const reserve = next + RESERVE_OFFSET + 2 * wave;
  put64(wcnt + WAVE_NEXT, uniform64(reserve[0]));
  put64(wcnt + WAVE_END, uniform64(reserve[1]));

  Lane<R> s;
  Lane<R> z;            // counters when this slice took the packet over
  SliceCount acc{0, 0, 0, 0, 0};
  int prob = 0;
  bool active = false;
  int fin = ST_NONE;     // status of a packet that has ended and is not recorded yet
  bool drained = false;
  uint32_t debt = 0;     // idle lane passes since the last refill
  {
    const SlotState &q = slots[gid];
    if (q.active) {
      load_slot<R>(q, s, &prob);
      const ProblemK &pb = probs[BATCH ? prob : 0];
      const int X[3] = {s.c.ox, s.c.oy, s.c.oz};
      locate(pb, X, stk, stride, s.c);
      s.lf = load_leaf<R>(pb.leaves, s.c.leaf);
      active = true;
      z = s;
    }
  }
  // A launch in which the queue runs dry ends one to two DRY_CHECKs later: with
  // more packets than lanes those that are left may be few, and the walkers take
  // them sooner (1.5e5 FP64 packets of 2000 events on 1.3e5 lanes: the last
  // 19e3 ran 16 ms alone in a launch of full length; the run 50.4 -> 43.8 ms).  A
  // run whose packets all start at once has no such moment, and short walks end
  // before the second look.  Where peel-off rays are walked inline there are no
  // walkers, and the packets walk faster spread out than gathered (a wave's step
  // lasts as long as its longest ray): 3e5 FP32 packets at tau 300, ended early 109
  // ms, in whole slices 78.
  int dry_at = DEFER && total > (int64_t)gridDim.x * blockDim.x && !queue_dry(next, total) ? 0 : -1;
  for (int it = 0; it < budget; ++it) {
    if (DEFER && *snk.count > room) break;
    if (DEFER && it % DRY_CHECK == DRY_CHECK - 1 && dry_at >= 0) {
      if (queue_dry(next, total)) {
        wcnt[WAVE_DRY] = it + 1;
        ++dry_at;
      }
      if (dry_at > 1) break;
    }
    // ---- record ended packets and refill idle lanes, together, once the
    // lanes have idled about as much as that costs the wave (REFILL_DEBT
    // lane passes), or none is active
    const unsigned long long idle = __ballot(!active);
    const uint32_t n_idle = (uint32_t)__popcll(idle);
    const bool all_idle = n_idle == 64u;
    debt += n_idle;
    if (all_idle || (!drained && debt >= REFILL_DEBT && (int)n_idle >= refill_min)) {
      debt = 0;
      if (fin != ST_NONE) {
        add_delta(acc, s, z);
        finish<R, BATCH>(probs[BATCH ? prob : 0], s, fin, wcnt + WAVE_ENDS, slice);
        fin = ST_NONE;
      }
      if (drained) break;
      // packets from the wave's reserve, then from the queue; one atomic
      // takes a wave's worth more than needed while the queue is long
      unsigned long long r_next = get64(wcnt + WAVE_NEXT), r_end = get64(wcnt + WAVE_END);
      const uint32_t have = (uint32_t)(r_end - r_next);
      unsigned long long base = r_next, lim = r_end;
      if (have < n_idle) {
        const unsigned long long ask = n_idle - have + (wcnt[WAVE_PLENTY] ? 64u : 0u);
        if (lane == 0) base = atomicAdd(next, ask);
        base = uniform64(base);
        if (base >= (unsigned long long)total) {
          drained = true;
          base = lim = (unsigned long long)total;
        } else {
          lim = (unsigned long long)total - base < ask ? (unsigned long long)total : base + ask;
          // (enough left for every wave to take more than it needs)
          wcnt[WAVE_PLENTY] = (unsigned long long)total - lim > (unsigned long long)gridDim.x * blockDim.x * 2u;
        }
      }
      const uint32_t rank = (uint32_t)__popcll(idle & ((1ull << lane) - 1ull));
      const unsigned long long g =
          have >= n_idle || rank < have ? r_next + rank : base + (rank - have);
      const bool take = !active && (rank < have || g < lim);
      wcnt[WAVE_STARTED] += __popcll(__ballot(take));
      if (have >= n_idle) {
        r_next += n_idle;
      } else {
        r_next = lim - base < n_idle - have ? lim : base + (n_idle - have);
        r_end = lim;
      }
      put64(wcnt + WAVE_NEXT, r_next);
      put64(wcnt + WAVE_END, r_end);
      if (take) {
        if (BATCH) {
          int lo = 0, hi = n_probs - 1;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (starts[mid] <= (int64_t)g) lo = mid; else hi = mid - 1;
          }
          prob = lo;
        }
        const ProblemK &pb = probs[BATCH ? prob : 0];
        const int64_t pid = pb.first + ((int64_t)g - starts[BATCH ? prob : 0]);
        emit<R, DEFER, NL>(pb, pid, s, stk, pstk, stride, snk);
        z = s;
        z.nscat = 0;
        z.cnt = LaneCount{0, 0, 0, 0, 0};
        int X[3];
        if (int_coords(pb.L, s.p, s.kd, X)) {
          locate(pb, X, stk, stride, s.c);
          s.lf = load_leaf<R>(pb.leaves, s.c.leaf);
          active = true;
        } else {
          fin = ST_ESCAPED;
        }
      }
    }
    if (!active) continue;

    const ProblemK &pb = probs[BATCH ? prob : 0];
    const double kd[3] = {s.kd[0], s.kd[1], s.kd[2]};
    Opac<R, NL> o;
    opacity(pb, s.lf, (double)s.x, s.k, o);
    double face[3], lo[3], hi[3];
    int em = 0;
    double te = 0.0, td = 0.0, lmax = 0.0, tseg = 0.0;
    // a pending line scattering (REGROUP) is already at its event point
    const bool pend = REGROUP && s.rej != 0;
    // An event closer than the nearest face of a leaf inside the domain
    // happens in this leaf whatever the exit distance; only a packet that
    // may leave needs it (the decision is the one tau < tseg would take).
    bool here = pend || (s.lf.bnd == R(0) && s.tau < (double)o.ktot * inner_dist(s.c, pb.L, s.p));
    if (here) {
      cell_bounds(s.c, pb.L, lo, hi);
    } else {
      te = exit_dist(s.c, pb.L, s.p, kd, face, lo, hi, &em);
      td = domain_dist_leaf(s.lf, pb.domain, pb.dom, s.p, kd);
      lmax = te < td ? te : td;
      tseg = (double)o.ktot * lmax;
      here = s.tau < tseg;
    }
    int st = ST_NONE;
    if (here) {
      // the event happens inside this leaf (float path: kappa is a float
      // and tau_event came from a float logarithm, so a float reciprocal
      // of kappa loses nothing the path keeps)
      // (a pending event moves by 0: p stays, clamped into its own leaf)
      const double dist = pend ? 0.0
                               : (sizeof(R) == 4 ? s.tau * (double)__builtin_amdgcn_rcpf((float)o.ktot)
                                                 : s.tau / (double)o.ktot);
#pragma unroll
      for (int d = 0; d < 3; ++d) s.p[d] = fmin(fmax(fma(dist, kd[d], s.p[d]), lo[d]), hi[d]);
      s.path += dist;
      if (!pend) ++s.event;
        if (!pend && pb.max_events > 0 && (int64_t)s.event >= pb.max_events) {
          st = ST_STUCK;
        } else {
          RngDraws<R, REGROUP> dr(pb, s);
          const StartCell<R> sc{&s.c, &s.lf, stk};
          st = interact<R, NL>(pb, s, o, dr, [&](const PeelSrc<R> &ps) {
            peel_all<R, DEFER, NL>(pb, s.p, ps, pstk, stride, s.cnt, snk, &sc);
          });
        }
    } else {
      s.tau -= tseg;
      s.path += lmax;
      ++s.cnt.cross;
      if (s.cnt.cross >= MAX_CROSS) {
        st = ST_STUCK;
      } else if (td <= te) {
#pragma unroll
        for (int d = 0; d < 3; ++d) s.p[d] = fma(td, kd[d], s.p[d]);
        st = ST_ESCAPED;
      } else {
        double pn[3];
        exit_point(te, em, s.p, kd, face, lo, hi, pn);
        s.p[0] = pn[0]; s.p[1] = pn[1]; s.p[2] = pn[2];
        wrap_slab(pb.domain, s.p, kd);
        int X[3];
        if (!int_coords(pb.L, s.p, kd, X)) {
          st = ST_ESCAPED;
        } else {
          relocate(pb, X, stk, stride, s.c);
          s.lf = load_leaf<R>(pb.leaves, s.c.leaf);
        }
      }
    }
    if (st != ST_NONE) {
      fin = st;
      active = false;
    }
  }
  if (fin != ST_NONE) {
    add_delta(acc, s, z);
    finish<R, BATCH>(probs[BATCH ? prob : 0], s, fin, wcnt + WAVE_ENDS, slice);
  }
  // ---- park the packet (if any) for the next launch, publish the counts
  SlotState &q = slots[gid];
  if (active) {
    save_slot<R>(q, s, prob);
    add_delta(acc, s, z);
  } else {
    q.active = 0;
  }
  if (queue && lane == 0) {
    pq->counts[wave] = (uint32_t)*snk.count;
  }
  if (lane == 0) {
    reserve[0] = get64(wcnt + WAVE_NEXT);
    reserve[1] = get64(wcnt + WAVE_END);
    if (wcnt[WAVE_STARTED]) atomicAdd(slice + N_STATS + 3, (unsigned long long)(uint32_t)wcnt[WAVE_STARTED]);
    // the length of a launch that ends on a dry queue
    if (DEFER && wcnt[WAVE_DRY]) atomicMax(slice + N_STATS + 4, (unsigned long long)wcnt[WAVE_DRY]);
  }
  publish(BATCH ? nullptr : probs[0].stats, acc, wcnt + WAVE_ENDS, slice);
}

// ------------------------------------------------- the last, longest walks
// Once every packet has started and the live ones are fewer than the chip's
// lanes at one wave per SIMD, a run's time is that of its longest walks, and
// a wave alone on its SIMD advances by about four cycles per instruction it
// issues, whether one of its lanes or all 64 take part.  k_walkers therefore
// gives a wave P = 2^lp packets (walker_waves picks P) and lets all its
// lanes work for them: in turns of 64/P loop passes,
//   - every lane computes the draws of one coming event of one packet (they
//     depend on the packet's index and the event's number alone), with the
//     functions that need nothing else (logarithms, sines, the phase
//     function's inverse), and leaves them in LDS;
//   - the P walking lanes run the passes on those draws and leave what an
//     event's peel-off needs in LDS;
//   - every lane runs the peel-off of one recorded event.
// The same expressions in the same order per packet as k_transport, so the
// same packets.  Cycles per event of 64 packets against k_transport
// (RMC_OPT_COMPACT 0): float 3480 against 6720 (slab, no observer) and 3620
// against 9000 (one observer), double 6540 / 16390 and 6840 / 21050.

// Columns of an event's draws in LDS ([column][64]).
enum {
  D_CHANNEL = 0, D_MU, D_LOG_TAU, D_SIN_PHI, D_COS_PHI, D_LOG_PERP, D_SIN_PERP, D_COS_PERP,
  D_REJ,                    // the first two rejection rounds: 2 x 3 (double) or 2 x 2 (float)
  D_MU_CORE = D_REJ + 6, D_MU_WING, D_DECAY, N_DRAWS
};

template <class R, int NL>
__device__ __forceinline__ void fill_draws(const ProblemK &pb, uint64_t pid, uint32_t event, R *col) {
  EventRng<R> rng(pb.seed, pid, event);
  col[D_CHANNEL * 64] = rng.u_small(J_CHANNEL);
  const R mu = rng.u(J_MU);
  col[D_MU * 64] = mu;
  col[D_MU_CORE * 64] = mu_dipole(mu, true);
  col[D_MU_WING * 64] = mu_dipole(mu, false);
  R sn, cs;
  M<R>::sincos2pi(rng.u(J_PHI), &sn, &cs);
  col[D_SIN_PHI * 64] = sn;
  col[D_COS_PHI * 64] = cs;
  col[D_LOG_TAU * 64] = M<R>::log(rng.u(J_TAU));
  // (float: the base-2 logarithm, scaled where it is used, as M<float>::log does)
  if constexpr (sizeof(R) == 4) col[D_LOG_PERP * 64] = __builtin_amdgcn_logf(rng.u(J_PERP1));
  else col[D_LOG_PERP * 64] = M<R>::log(rng.u(J_PERP1));
  M<R>::sincos2pi(rng.u(J_PERP2), &sn, &cs);
  col[D_SIN_PERP * 64] = sn;
  col[D_COS_PERP * 64] = cs;
  constexpr int n = sizeof(R) == 8 ? 6 : 4;
#pragma unroll
  for (int j = 0; j < n; ++j) col[(D_REJ + j) * 64] = rng.u(J_REJ + j);
  if constexpr (NL > 1) {
    bool fluor = false;
#pragma unroll
    for (int q = 0; q < NL; ++q) fluor = fluor || (q < pb.n_lines && pb.lines[q].n_fluor > 0);
    if (fluor) col[D_DECAY * 64] = rng.u(J_DECAY);
  }
}

// The draws of one event from their columns, as interact takes them.
template <class R, int NL> struct LdsDraws {
  uint64_t seed;
  R v[N_DRAWS];
  __device__ __forceinline__ LdsDraws(uint64_t sd, const R *col) : seed(sd) {
#pragma unroll
    for (int j = 0; j < N_DRAWS; ++j)
      if ((j < D_REJ || j >= D_MU_CORE || j < D_REJ + (sizeof(R) == 8 ? 6 : 4)) && (NL > 1 || j != D_DECAY))
        v[j] = col[j * 64];
  }
  __device__ __forceinline__ R channel() const { return v[D_CHANNEL]; }
  __device__ __forceinline__ R albedo() const { return v[D_REJ]; }   // J_ALBEDO is the first round's first draw
  __device__ __forceinline__ R mu() const { return v[D_MU]; }
  __device__ __forceinline__ R log_tau() const { return v[D_LOG_TAU]; }
  __device__ __forceinline__ void line() const {}
  __device__ __forceinline__ R log_perp() const {
    return sizeof(R) == 4 ? v[D_LOG_PERP] * R(0.69314718055994531) : v[D_LOG_PERP];
  }
  __device__ __forceinline__ void perp(R *sp, R *cp) const { *sp = v[D_SIN_PERP]; *cp = v[D_COS_PERP]; }
  __device__ __forceinline__ void phi(R *sp, R *cp) const { *sp = v[D_SIN_PHI]; *cp = v[D_COS_PHI]; }
  __device__ __forceinline__ void phi_dust(R *sp, R *cp) const { phi(sp, cp); }
  __device__ __forceinline__ R decay() const { return v[D_DECAY]; }
  __device__ __forceinline__ R dipole(bool core) const { return core ? v[D_MU_CORE] : v[D_MU_WING]; }
  __device__ __forceinline__ bool round(const UparEnv<R> &e, R a, int it, R *out) const {
    if constexpr (sizeof(R) == 4) return upar_try_pair(e, a, v[D_REJ + 2 * it], v[D_REJ + 2 * it + 1], out);
    else return upar_try_triple(e, a, v[D_REJ + 3 * it], v[D_REJ + 3 * it + 1], v[D_REJ + 3 * it + 2], out);
  }
  // From round s.rej on (not 0 for an event that a regrouped launch left
  // pending); the rounds beyond the second draw their own numbers.
  __device__ __forceinline__ bool upar(Lane<R> &s, R x, R a, R la, R *out) const {
    uint32_t it = s.rej;
    s.rej = 0;
    if (fabs(x) >= R(8)) {
      *out = upar_gauss<R>(x, v[D_REJ], v[D_REJ + 1]);
      return true;
    }
    const UparEnv<R> e = upar_env(x, a, la);
    if (it == 0 && round(e, a, 0, out)) return true;
    if (it <= 1 && round(e, a, 1, out)) return true;
    EventRng<R> rng(seed, (uint64_t)s.pid, s.event);
    for (it = it < 2 ? 2 : it; it < MAX_REJECT; ++it)
      if (upar_try(e, a, rng, it, out)) return true;
    return false;
  }
  static __device__ __forceinline__ int undrawn(Lane<R> &) { return ST_STUCK; }
};

// What an event's peel-off needs, in LDS ([column][64]): the event's point,
// its source (direction in, frequency, atom velocity; dust keeps k_in . u in
// the first velocity) and its cell.
template <class R> struct PeelCols {
  double p[3 * 64];
  R v[7 * 64];       // k_in, x, U
  int i[6 * 64];     // kind | line << 4 | core << 8 (-1: none), leaf, level, origin
};

template <class R>
__device__ __forceinline__ void record_peel(PeelCols<R> &c, int j, const Lane<R> &s, const PeelSrc<R> &ps) {
  const bool dust = ps.kind == 2;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    c.p[d * 64 + j] = s.p[d];
    c.v[d * 64 + j] = ps.kin[d];
  }
  c.v[3 * 64 + j] = ps.x;
  c.v[4 * 64 + j] = dust ? ps.w : ps.U[0];
  if (!dust) {
    c.v[5 * 64 + j] = ps.U[1];
    c.v[6 * 64 + j] = ps.U[2];
  }
  c.i[j] = dust ? ps.kind : ps.kind | (ps.line << 4) | (ps.core << 8);
  c.i[64 + j] = s.c.leaf;
  c.i[2 * 64 + j] = s.c.level;
  c.i[3 * 64 + j] = s.c.ox;
  c.i[4 * 64 + j] = s.c.oy;
  c.i[5 * 64 + j] = s.c.oz;
}

template <class R, int NL>
__device__ __forceinline__ void peel_recorded(const ProblemK &pb, const PeelCols<R> &c, int j, LaneCount &cnt,
                                              const PeelSink<R> &snk) {
  const int code = c.i[j];
  PeelSrc<R> ps;
  ps.kind = code & 15;
  ps.line = (code >> 4) & 15;
  ps.core = code >> 8;
  const double p[3] = {c.p[j], c.p[64 + j], c.p[2 * 64 + j]};
  const Cell cell{c.i[64 + j], c.i[2 * 64 + j], c.i[3 * 64 + j], c.i[4 * 64 + j], c.i[5 * 64 + j]};
  const LeafRec<R> lf = load_leaf<R>(pb.leaves, cell.leaf);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    ps.kin[d] = c.v[d * 64 + j];
    ps.U[d] = c.v[(4 + d) * 64 + j];
  }
  ps.x = c.v[3 * 64 + j];
  ps.w = ps.U[0];
  ps.ux = lf.ux; ps.uy = lf.uy; ps.uz = lf.uz;
  ps.irho = lf.irho;
  ps.rho = M<R>::div(R(1), lf.irho);
  const LineK &ln = pb.lines[ps.kind == 2 ? 0 : ps.line];
  ps.bc = cst<R>(pb.b_ref, pb.b_ref_f) * cst<R>(ln.mu, ln.f.mu) * ps.rho;
  const StartCell<R> sc{&cell, &lf, nullptr};
  peel_all<R, true, NL>(pb, p, ps, nullptr, 0, cnt, snk, &sc);
}

// One wave per block; wave w walks slots [w P, w P + P), all of one problem,
// and queues peel-off rays in region region0 + w.
template <class R, bool BATCH, int NL>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 1)))
    k_walkers(const ProblemK *__restrict__ probs, int region0, SlotState *__restrict__ slots, int lp, int budget,
              unsigned long long *__restrict__ slice) {
  extern __shared__ int lds[];
  __shared__ R draws[N_DRAWS * 64];
  __shared__ PeelCols<R> rec;
  __shared__ int walker_cnt[3 * 64];   // peel-off rays, leaves crossed and dropped deposits of each walker's turn
  __shared__ int wcnt[4];              // queued rays, then the packets that escaped, were absorbed, got stuck
  const int lane = threadIdx.x;
  const int P = 1 << lp, K = 64 >> lp;
  int *stk = lds + lane;
  Lane<R> s, z;
  SliceCount acc{0, 0, 0, 0, 0};
  int prob = 0, fin = ST_NONE;
  bool active = false;
  SlotState &q = slots[(int64_t)blockIdx.x * P + (lane & (P - 1))];
  if (lane < P && q.active) {
    load_slot<R>(q, s, &prob);
    active = true;
  }
  if (lane < 4) wcnt[lane] = 0;
  for (int j = lane; j < 3 * 64; j += 64) walker_cnt[j] = 0;
  PeelQueue *const pq = probs[0].pq;
  const bool queue = pq != nullptr;
  const int region = region0 + (int)blockIdx.x;
  const unsigned long long live = __ballot(active);
  if (live == 0ull) {
    if (queue && lane == 0) pq->counts[region] = 0u;
    return;
  }
  if (BATCH) prob = __builtin_amdgcn_readfirstlane(__shfl(prob, __ffsll((long long)live) - 1));
  const ProblemK &pb = probs[BATCH ? prob : 0];
  __shared__ LineK lines[NL];
  if (NL > 1) {
    for (int j = lane; j < (int)(NL * sizeof(LineK) / 4); j += 64) ((uint32_t *)lines)[j] = ((const uint32_t *)pb.lines)[j];
  }
  const WalkK<NL> wk(pb, lines);
  if (active) {
    const int X[3] = {s.c.ox, s.c.oy, s.c.oz};
    locate(wk, X, stk, 64, s.c);
    s.lf = load_leaf<R>(wk.leaves, s.c.leaf);
    z = s;
    if (s.rej) --s.event;   // a pending event is taken up again as the next one
  }
  PeelSink<R> snk;
  snk.count = wcnt;
  snk.region = queue ? (PeelJob<R> *)pq->jobs + (size_t)region * pq->cap : nullptr;
  snk.cap = queue ? (uint32_t)pq->cap : 0u;
  snk.lost = queue ? &pq->lost : nullptr;
  const int room = queue ? (int)pq->cap - 64 * MAX_OBS : 0x7fffffff;
  __syncthreads();
  for (int it = 0; it < budget; it += K) {
    const unsigned long long walking = __ballot(active);
    if (walking == 0ull || wcnt[0] > room) break;
    // ---- the draws of the coming events, one per lane
    {
      const int w = lane & (P - 1);
      const uint32_t plo = (uint32_t)__shfl((int)(uint32_t)s.pid, w), phi = (uint32_t)__shfl((int)(uint32_t)(s.pid >> 32), w);
      const uint32_t ev = (uint32_t)__shfl((int)s.event, w);
      if ((walking >> w) & 1ull)
        fill_draws<R, NL>(pb, (uint64_t)phi << 32 | plo, ev + 1u + (uint32_t)(lane >> lp), draws + lane);
      rec.i[lane] = -1;
    }
    __syncthreads();
    // ---- the walkers' passes
    const int turn = budget - it < K ? budget - it : K;
    int used = lane;   // this lane's next column of draws
    for (int b = 0; active && b < turn; ++b) {
      Opac<R, NL> o;
      opacity(wk, s.lf, (double)s.x, s.k, o);
      double face[3], lo[3], hi[3];
      int em = 0;
      double te = 0.0, td = 0.0, lmax = 0.0, tseg = 0.0;
      const bool pend = s.rej != 0;
      bool here = pend || (s.lf.bnd == R(0) && s.tau < (double)o.ktot * inner_dist(s.c, wk.L, s.p));
      if (here) {
        cell_bounds(s.c, wk.L, lo, hi);
      } else {
        te = exit_dist(s.c, wk.L, s.p, s.kd, face, lo, hi, &em);
        td = domain_dist_leaf(s.lf, wk.domain, wk.dom, s.p, s.kd);
        lmax = te < td ? te : td;
        tseg = (double)o.ktot * lmax;
        here = s.tau < tseg;
      }
      int st = ST_NONE;
      if (here) {
        const double dist = pend ? 0.0
                                 : (sizeof(R) == 4 ? s.tau * (double)__builtin_amdgcn_rcpf((float)o.ktot)
                                                   : s.tau / (double)o.ktot);
#pragma unroll
        for (int d = 0; d < 3; ++d) s.p[d] = fmin(fmax(fma(dist, s.kd[d], s.p[d]), lo[d]), hi[d]);
        s.path += dist;
        ++s.event;
        if (!pend && wk.max_events > 0 && (int64_t)s.event >= wk.max_events) {
          st = ST_STUCK;
        } else {
          LdsDraws<R, NL> dr(wk.seed, draws + used);
          st = interact<R, NL>(wk, s, o, dr, [&](const PeelSrc<R> &ps) { record_peel(rec, used, s, ps); });
          used += P;
        }
      } else {
        s.tau -= tseg;
        s.path += lmax;
        ++s.cnt.cross;
        if (s.cnt.cross >= MAX_CROSS) {
          st = ST_STUCK;
        } else if (td <= te) {
#pragma unroll
          for (int d = 0; d < 3; ++d) s.p[d] = fma(td, s.kd[d], s.p[d]);
          st = ST_ESCAPED;
        } else {
          double pn[3];
          exit_point(te, em, s.p, s.kd, face, lo, hi, pn);
          s.p[0] = pn[0]; s.p[1] = pn[1]; s.p[2] = pn[2];
          wrap_slab(wk.domain, s.p, s.kd);
          int X[3];
          if (!int_coords(wk.L, s.p, s.kd, X)) {
            st = ST_ESCAPED;
          } else {
            relocate(wk, X, stk, 64, s.c);
            s.lf = load_leaf<R>(wk.leaves, s.c.leaf);
          }
        }
      }
      if (st != ST_NONE) {
        fin = st;
        active = false;
      }
    }
    __syncthreads();
    // ---- the peel-off of the turn's events, one per lane
    if (wk.n_obs) {
      if (rec.i[lane] >= 0) {
        LaneCount c{0, 0, 0, 0, 0};
        peel_recorded<R, NL>(pb, rec, lane, c, snk);
        const int w = lane & (P - 1);
        atomicAdd(walker_cnt + w, (int)c.peel_rays);
        if (c.peel_cross) atomicAdd(walker_cnt + 64 + w, (int)c.peel_cross);
        if (c.peel_drop) atomicAdd(walker_cnt + 128 + w, (int)c.peel_drop);
      }
      __syncthreads();
      if (lane < P) {
        s.cnt.peel_rays += (uint32_t)walker_cnt[lane];
        s.cnt.peel_cross += (uint32_t)walker_cnt[64 + lane];
        s.cnt.peel_drop += (uint32_t)walker_cnt[128 + lane];
        walker_cnt[lane] = walker_cnt[64 + lane] = walker_cnt[128 + lane] = 0;
      }
    }
    if (fin != ST_NONE) {
      add_delta(acc, s, z);
      finish<R, BATCH>(pb, s, fin, wcnt + 1, slice);
      fin = ST_NONE;
      if (lane < P) q.active = 0;
    }
    __syncthreads();
  }
  if (active) {
    if (s.rej) ++s.event;   // not reached: still pending
    save_slot<R>(q, s, prob);
    add_delta(acc, s, z);
  }
  if (queue && lane == 0) pq->counts[region] = (uint32_t)wcnt[0];
  publish(BATCH ? nullptr : pb.stats, acc, wcnt + 1, slice);
}

// Number of slots (lanes) holding a packet after a launch.
__global__ void k_count_live(const SlotState *__restrict__ slots, int64_t n, unsigned long long *out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned long long v = (i < n && slots[i].active) ? 1ull : 0ull;
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
  if (__lane_id() == 0 && v) atomicAdd(out, v);
}

__global__ void k_clear_slots(SlotState *__restrict__ slots, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) slots[i].active = 0;
}

// Parked packets gathered to the front: every active slot of src[0, n) is
// copied to its own slot of dst (order not kept; a packet's walk does not
// depend on the lane that runs it), one atomic per wave; *n_live counts
// them.  Once every packet of a stream has started, the launches that
// follow run on the gathered slots with as many waves as the packets fill,
// so the last long walks share fewer SIMDs and each wave issues faster.
__global__ void k_compact_slots(const SlotState *__restrict__ src, int64_t n, SlotState *__restrict__ dst,
                                unsigned long long *n_live) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool act = i < n && src[i].active;
  const unsigned long long m = __ballot(act);
  if (m == 0ull) return;
  const int lane = __lane_id();
  const int leader = __ffsll((long long)m) - 1;
  unsigned long long base = 0;
  if (lane == leader) base = atomicAdd(n_live, (unsigned long long)__popcll(m));
  base = __shfl(base, leader);
  if (act) dst[base + (unsigned long long)__popcll(m & ((1ull << lane) - 1ull))] = src[i];
}

// The same for a batch, each problem's packets in slots of their own, a
// multiple of P of them, so that every wave of k_walkers holds packets of one
// problem: work[p] counts problem p's live packets (k_group_count), becomes
// its first slot (k_group_offsets), then its next free one (k_group_slots).
__global__ void k_group_count(const SlotState *__restrict__ src, int64_t n, uint32_t *work) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && src[i].active) atomicAdd(work + src[i].prob, 1u);
}

__global__ void __launch_bounds__(1024) k_group_offsets(uint32_t *work, int n_probs, int lp,
                                                        unsigned long long *n_live) {
  __shared__ uint32_t part[16];
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  uint32_t base = 0, live = 0;
  for (int b = 0; b < n_probs; b += 1024) {
    const int p = b + (int)threadIdx.x;
    const uint32_t c = p < n_probs ? work[p] : 0u;
    const uint32_t v = ((c + (1u << lp) - 1u) >> lp) << lp;
    live += c;
    uint32_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(x, off);
      if (lane >= off) x += y;
    }
    if (lane == 63) part[wave] = x;
    __syncthreads();
    uint32_t before = base, all = base;
    for (int w = 0; w < 16; ++w) {
      if (w < wave) before += part[w];
      all += part[w];
    }
    if (p < n_probs) work[p] = before + x - v;
    base = all;
    __syncthreads();
  }
  for (int off = 32; off > 0; off >>= 1) live += __shfl_xor(live, off);
  if (lane == 0 && live) atomicAdd(n_live, (unsigned long long)live);
}

__global__ void k_group_slots(const SlotState *__restrict__ src, int64_t n, SlotState *__restrict__ dst, int64_t n_dst,
                              uint32_t *work) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || !src[i].active) return;
  const int64_t j = atomicAdd(work + src[i].prob, 1u);
  if (j < n_dst) dst[j] = src[i];
}

// Before the ray-cast pass: offs[r] = jobs queued in regions 0 .. r - 1 of the
// launch's n_regions waves, so that the pass can hand out its jobs by one
// running index whatever the regions hold.  Reports the launch's pushes, its
// fullest region and its lost pushes (slice counters N_STATS .. N_STATS + 2)
// and resets the queue's totals.  One block: a few thousand counts.
__global__ void __launch_bounds__(1024) k_peel_scan(PeelQueue *pq, int n_regions, unsigned long long *slice) {
  __shared__ uint32_t part[16], top[16];
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  const uint32_t cap = (uint32_t)pq->cap;
  uint32_t base = 0, most = 0;
  for (int b = 0; b < n_regions; b += 1024) {
    const int r = b + (int)threadIdx.x;
    const uint32_t c = r < n_regions ? pq->counts[r] : 0u;
    most = c > most ? c : most;
    const uint32_t v = c < cap ? c : cap;
    uint32_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(x, off);
      if (lane >= off) x += y;
    }
    if (lane == 63) part[wave] = x;
    __syncthreads();
    uint32_t before = base, all = base;
    for (int w = 0; w < 16; ++w) {
      if (w < wave) before += part[w];
      all += part[w];
    }
    if (r < n_regions) pq->offs[r] = before + x - v;
    base = all;
    __syncthreads();
  }
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t y = __shfl_xor(most, off);
    most = y > most ? y : most;
  }
  if (lane == 0) top[wave] = most;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) most = top[w] > most ? top[w] : most;
    pq->offs[n_regions] = base;
    pq->n_regions = (unsigned long long)n_regions;
    slice[N_STATS] = base;
    slice[N_STATS + 1] = most;
    slice[N_STATS + 2] = pq->lost;
    pq->lost = 0ull;
    pq->take = 0ull;
  }
}

// The region holding queued job j: the last r with offs[r] <= j (j < offs[n]).
// The wave's lanes test 64 regions at a time, so 4096 regions take two loads.
__device__ __forceinline__ uint32_t region_of(const uint32_t *__restrict__ offs, uint32_t n, uint32_t j, int lane) {
  uint32_t lo = 0;
  while (n > 1) {
    const uint32_t step = (n + 63) / 64;
    const uint32_t i = (uint32_t)lane * step;
    const unsigned long long m = __ballot(i < n && offs[lo + i] <= j);
    const uint32_t k = (uint32_t)(__popcll(m) - 1) * step;
    lo += k;
    n = n - k < step ? n - k : step;
  }
  return lo;
}

// --------------------------------------------------------- rays, leaf by leaf
// A ray of fixed direction walked one leaf per step.  The next leaf's record is
// asked for before the current one's opacity is computed: the geometry does not
// depend on the record, so its load is hidden by that arithmetic (a ray is a
// chain of dependent reads, and few rays leave nothing else to hide them).
// The distances are the correctly rounded quotients of exit_dist or, on the float
// image path, its products with 1/k.  With AXIS the axes a direction does not move
// along are branched round; without, all three are computed without a branch, so
// that their chains overlap: behind branches of their own they ran one after
// another, and oblique rays were slower than with divisions.
// Measured in us: walks that divide, without the early load and with the lines in
// a loop -> branched -> now.  FP64 images along (1,1,1), one line, 6e4 rays 233 ->
// 227 -> 190, 4e6 rays 3759 -> 4031 -> 3258; two lines, 4e6 rays 2661 -> 3026 ->
// 2567; FP32, 6e4 rays 187 -> 177 -> 143.  FP64 along z with crossing lists, 3e5 rays
// 267 -> 235 (AXIS).
template <class R, bool PRODUCT, bool AXIS> struct RayWalk {
  double p[3];
  int X[3];
  Cell c;
  LeafRec<R> lf;
  bool by_quotient;

  // The leaf of p; false outside the unit cube.
  template <class PB>
  __device__ __forceinline__ bool start(const PB &pb, const double k[3], int *stk, int stride) {
    if (!int_coords(pb.L, p, k, X)) return false;
    by_quotient = quotient_holds(p, k);
    locate(pb, X, stk, stride, c);
    lf = load_leaf<R>(pb.leaves, c.leaf);
    return true;
  }

  // Leaves leaf *leaf (segment *seg, record *rec) for the next one; false when
  // the ray ends at the domain border or leaves the cube.
  template <class PB>
  __device__ __forceinline__ bool step(const PB &pb, const double k[3], const double kinv[3], int *stk, int stride,
                                       int *leaf, double *seg, LeafRec<R> *rec) {
    const double inv = ldexp(1.0, -pb.L), sc = (double)(1 << pb.L);
    const int side = 1 << pb.L, sz = 1 << (pb.L - c.level);
    const int o[3] = {c.ox, c.oy, c.oz};
    double lo[3], hi[3], t[3], te = __builtin_inf();
    double pn[3] = {p[0], p[1], p[2]};
    bool in = true;
    int Y[3] = {X[0], X[1], X[2]};
    if constexpr (AXIS) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        t[d] = __builtin_inf();
        if (k[d] != 0.0) {
          lo[d] = (double)o[d] * inv;
          hi[d] = (double)(o[d] + sz) * inv;
          const double a = (k[d] > 0.0 ? hi[d] : lo[d]) - p[d];
          t[d] = PRODUCT ? a * kinv[d] : (by_quotient ? quotient(a, k[d], kinv[d]) : a / k[d]);
          te = t[d] < te ? t[d] : te;
        }
      }
      te = te < 0.0 ? 0.0 : te;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        if (k[d] != 0.0) {
          const double q = fmin(fmax(fma(te, k[d], p[d]), lo[d]), hi[d]);
          pn[d] = t[d] <= te ? (k[d] > 0.0 ? hi[d] : lo[d]) : q;
        }
      }
      wrap_slab(pb.domain, pn, k);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        if (k[d] != 0.0) {
          const double s = pn[d] * sc;
          const double f = k[d] > 0.0 ? floor(s) : ceil(s) - 1.0;
          const bool ok = f >= 0.0 && f < (double)side;
          in = in && ok;
          Y[d] = ok ? (int)f : 0;
        }
      }
    } else {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        lo[d] = (double)o[d] * inv;
        hi[d] = (double)(o[d] + sz) * inv;
        t[d] = (k[d] > 0.0 ? hi[d] : lo[d]) - p[d];
      }
      if (PRODUCT) {
#pragma unroll
        for (int d = 0; d < 3; ++d) t[d] *= kinv[d];
      } else if (by_quotient) {
#pragma unroll
        for (int d = 0; d < 3; ++d) t[d] = quotient(t[d], k[d], kinv[d]);
      } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) t[d] /= k[d];
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        t[d] = k[d] != 0.0 ? t[d] : __builtin_inf();
        te = t[d] < te ? t[d] : te;
      }
      te = te < 0.0 ? 0.0 : te;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double q = fmin(fmax(fma(te, k[d], p[d]), lo[d]), hi[d]);
        pn[d] = t[d] <= te ? (k[d] > 0.0 ? hi[d] : lo[d]) : q;
      }
      wrap_slab(pb.domain, pn, k);
      in = int_coords(pb.L, pn, k, Y);
    }
    *leaf = c.leaf;
    *rec = lf;
    const double td = domain_dist_leaf(lf, pb.domain, pb.dom, p, k);
    *seg = td <= te ? td : te;
    if (!in || td <= te) return false;
    relocate(pb, Y, stk, stride, c);
    lf = load_leaf<R>(pb.leaves, c.leaf);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      p[d] = pn[d];
      if (AXIS) X[d] = Y[d];
    }
    return true;
  }
};

// Ray-cast pass over the peel-off rays queued by a transport launch.  A
// wave takes runs of queued jobs by their running index over all regions
// (k_peel_scan), so the pass spreads over the chip also where a few waves
// queued every ray, as at the end of a run (handing a wave a whole region
// left a complete 2e5-packet run of the dusty sphere at tau0 = 5e3 with
// 208 ms of this pass, now 42); each lane
// walks one ray a leaf per iteration and takes the run's next ray as soon as
// its own is done, so the waves stay full while ray lengths vary.  The walk starts from
// the queued state (a ray's start, or where it left its first leaf), and every
// deferred deposit is made here.
// Bound by the latency of its loads with four waves on a SIMD (vector
// instructions take half the cycles; five waves spill).  RayWalk's early load
// and a problem kept in registers gave 2%.  ONE, for a run of one problem and one
// observer: the direction is the launch's, so it stays in scalar registers, and
// the axes it does not move along cost nothing.  The pass in ms, general ->
// ONE: dusty sphere 5e5 FP32 packets 16.5 -> 13.0, 2e5 to their end 42.0 -> 32.0,
// H + D 18 -> 12.7, 1.5e5 FP64 packets 4.45 -> 4.13.
#ifndef RMC_DRAIN_WAVES_F32
#define RMC_DRAIN_WAVES_F32 4
#endif
#ifndef RMC_DRAIN_WAVES_F64
#define RMC_DRAIN_WAVES_F64 3
#endif
template <class R> struct DrainWaves;
template <> struct DrainWaves<float> { static constexpr int v = RMC_DRAIN_WAVES_F32; };
template <> struct DrainWaves<double> { static constexpr int v = RMC_DRAIN_WAVES_F64; };

template <class R, bool BATCH, bool ONE, int NL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DrainWaves<R>::v)))
    k_peel_drain(const ProblemK *__restrict__ probs, PeelQueue *pq,
                                                    unsigned long long *__restrict__ slice) {
  extern __shared__ int lds[];
  const int stride = blockDim.x;
  int *stk = lds + threadIdx.x;
  const int lane = __lane_id();
  const unsigned long long cap = pq->cap;
  const uint32_t n_regions = (uint32_t)pq->n_regions;
  const PeelJob<R> *__restrict__ jobs = (const PeelJob<R> *)pq->jobs;
  const uint32_t *__restrict__ offs = pq->offs;
  const uint32_t total = offs[n_regions];
  // jobs a wave takes at once: enough to spread what the take and its
  // region search cost, few enough that the waves end together
  const uint32_t share = total / (gridDim.x * (blockDim.x / 64) * 8u);
  const uint32_t run = share < 64u ? 64u : (share > 1024u ? 1024u : share);
  const double cut = TauCut<R>::v;
  // wave-uniform: next job and end of the wave's run (its first one by its
  // index, the next ones from pq->take), the region of the next job, its first
  // job and its end (running indices)
  const uint32_t wave = (uint32_t)blockIdx.x * (blockDim.x / 64) + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t waves = gridDim.x * (blockDim.x / 64);
  if ((unsigned long long)wave * run >= total) return;
  uint32_t cur = wave * run, end = total - cur < run ? total : cur + run, reg = 0, r_beg = 0, r_end = 0;
  bool drained = false;
  bool active = false;
  int prob = 0, acc_prob = 0;
  const WalkK<NL> one(probs[0], nullptr);   // the problem of a run without a batch, in registers
  double k[3], kinv[3], tau = 0.0, x = 0.0;
  R weight = R(0), kr[3];
  if constexpr (ONE) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      k[d] = probs[0].obs[0].k[d];
      kinv[d] = probs[0].obs[0].kinv[d];
      kr[d] = (R)k[d];
    }
  }
  unsigned long long elem = 0;
  int oi = 0;
  uint32_t steps = 0;
  RayWalk<R, sizeof(R) == 4, true> wk;   // (AXIS: 3% faster along z, 3-5% slower along (1,1,1))
  unsigned long long nc_prob = 0, nc_all = 0;
  unsigned long long nd_prob = 0, nd_all = 0;   // float jobs outside the cube
  while (true) {
    unsigned long long idle = __ballot(!active);
    while (idle && !drained) {
      if (cur >= end) {
        unsigned long long t = 0;
        if (lane == 0) t = atomicAdd(&pq->take, (unsigned long long)run);
        t = __shfl(t, 0) + (unsigned long long)waves * run;
        if (t >= total) {
          drained = true;
          break;
        }
        cur = (uint32_t)t;
        end = total - cur < run ? total : cur + run;
        r_end = 0;
      }
      if (cur >= r_end) {
        reg = region_of(offs, n_regions, cur, lane);
        r_beg = offs[reg];
        r_end = offs[reg + 1];
      }
      const uint32_t avail = (end < r_end ? end : r_end) - cur;
      const uint32_t rank = (uint32_t)__popcll(idle & ((1ull << lane) - 1ull));
      const bool mine = ((idle >> lane) & 1ull) && rank < avail;
      if (mine) {
        const PeelJob<R> j = jobs[reg * cap + (cur - r_beg) + rank];
        const int jp = BATCH ? (int)(j.dst >> PQ_PROB_SHIFT) : 0;
        if (BATCH && jp != acc_prob) {
          if (nc_prob) atomicAdd(probs[acc_prob].stats + S_PEEL_CROSS, nc_prob);
          if (nd_prob) atomicAdd(probs[acc_prob].stats + S_PEEL_DROPPED, nd_prob);
          nc_prob = 0;
          nd_prob = 0;
          acc_prob = jp;
        }
        prob = jp;
        const ProblemK &pb = probs[prob];
        oi = ONE ? 0 : (int)((j.dst >> PQ_OBS_SHIFT) & 15ull);
        const ObsK &ob = pb.obs[oi];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          wk.p[d] = j.p[d];
          if constexpr (!ONE) {
            k[d] = ob.k[d];
            kinv[d] = ob.kinv[d];
            kr[d] = (R)k[d];
          }
        }
        x = (double)j.x;
        weight = (R)j.weight;
        bool binned = true;
        if constexpr (sizeof(R) == 8) {
          tau = j.tau;
          steps = j.steps;
          elem = j.dst & PQ_ELEM_MASK;
        } else {
          // float jobs come unbinned, from the ray's start
          tau = 0.0;
          steps = 0;
          const int pix = pixel_of<true>(ob, wk.p);
          const int bin = bin_of<true>(ob, x);
          binned = pix >= 0 && bin >= 0;
          elem = binned ? (unsigned long long)pix * ob.nbins + bin : 0ull;
          if (!binned) {
            ++nd_prob;
            ++nd_all;
          }
        }
        if (binned) {
          if (steps < MAX_CROSS) active = BATCH ? wk.start(pb, k, stk, stride) : wk.start(one, k, stk, stride);
          if (!active && tau < cut)
            atomic_add_real((R *)ob.cube + elem, weight * M<R>::exp((R)(-tau)));
        }
      }
      const uint32_t n_idle = (uint32_t)__popcll(idle);
      cur += avail < n_idle ? avail : n_idle;
      // lanes given a job that ended at once stay idle until the next pass
      idle &= ~__ballot(mine);
    }
    if (__ballot(active) == 0ull) {
      if (drained) break;
      continue;
    }
    if (!active) continue;
    int leaf;
    double seg;
    LeafRec<R> lf;
    Opac<R, NL> o;
    if constexpr (BATCH) {
      active = wk.step(probs[prob], k, kinv, stk, stride, &leaf, &seg, &lf);
      opacity(probs[prob], lf, x, kr, o);
    } else {
      active = wk.step(one, k, kinv, stk, stride, &leaf, &seg, &lf);
      opacity(one, lf, x, kr, o);
    }
    ++nc_prob;
    ++nc_all;
    tau += (double)o.ktot * seg;
    if (tau >= cut || ++steps >= MAX_CROSS) active = false;
    if (!active && tau < cut)
      atomic_add_real((R *)probs[prob].obs[oi].cube + elem, weight * M<R>::exp((R)(-tau)));
  }
  // crossings and dropped deposits: per problem, and for the launch's
  // slice counters
  if (BATCH) {
    if (nc_prob) atomicAdd(probs[acc_prob].stats + S_PEEL_CROSS, nc_prob);
    if (nd_prob) atomicAdd(probs[acc_prob].stats + S_PEEL_DROPPED, nd_prob);
  } else {
    unsigned long long v = nc_prob, d = nd_prob;
    for (int off = 32; off > 0; off >>= 1) {
      v += __shfl_down(v, off);
      d += __shfl_down(d, off);
    }
    if (lane == 0 && v) atomicAdd(probs[0].stats + S_PEEL_CROSS, v);
    if (lane == 0 && d) atomicAdd(probs[0].stats + S_PEEL_DROPPED, d);
  }
  unsigned long long v = nc_all, d = nd_all;
  for (int off = 32; off > 0; off >>= 1) {
    v += __shfl_down(v, off);
    d += __shfl_down(d, off);
  }
  if (lane == 0 && v) atomicAdd(slice + S_PEEL_CROSS, v);
  if (lane == 0 && d) atomicAdd(slice + S_PEEL_DROPPED, d);
}

// ---------------------------------------------------------- optical depths
// Optical depth of the ray from p0 along k to the domain border; stops once
// it reaches tau_cut.
template <class R, int NL, bool PRODUCT, bool AXIS>
__device__ __forceinline__ double walk_tau(const ProblemK &pb, const double p0[3], const double k[3],
                                           const double kinv[3], double x_ext, double tau_cut, int *stk, int stride,
                                           uint32_t *ncross) {
  const R kr[3] = {(R)k[0], (R)k[1], (R)k[2]};
  RayWalk<R, PRODUCT, AXIS> w;
  w.p[0] = p0[0]; w.p[1] = p0[1]; w.p[2] = p0[2];
  double tau = 0.0;
  bool more = w.start(pb, k, stk, stride);
  while (more) {
    int leaf;
    double seg;
    LeafRec<R> rec;
    more = w.step(pb, k, kinv, stk, stride, &leaf, &seg, &rec);
    Opac<R, NL> o;
    opacity(pb, rec, x_ext, kr, o);
    tau += (double)o.ktot * seg;
    ++*ncross;
    if (tau >= tau_cut || *ncross >= MAX_CROSS) break;
  }
  return tau;
}

// ------------------------------------------------------------------ probes
__global__ void k_trace(ProblemK pb, int64_t n, const double *__restrict__ orig,
                        const double *__restrict__ dir, int max_cells, int32_t *__restrict__ leaf_out,
                        double *__restrict__ seg_out, int32_t *__restrict__ n_out) {
  extern __shared__ int lds[];
  int *stk = lds + threadIdx.x;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  double p[3] = {orig[3 * r], orig[3 * r + 1], orig[3 * r + 2]};
  const double k[3] = {dir[3 * r], dir[3 * r + 1], dir[3 * r + 2]};
  int X[3];
  int cnt = 0;
  if (int_coords(pb.L, p, k, X)) {
    Cell c;
    locate(pb, X, stk, blockDim.x, c);
    while (cnt < max_cells) {
      double face[3], lo[3], hi[3];
      int em;
      const double te = exit_dist(c, pb.L, p, k, face, lo, hi, &em);
      const double td = domain_dist(pb.domain, pb.dom, p, k);
      leaf_out[r * max_cells + cnt] = c.leaf;
      if (td <= te) {
        seg_out[r * max_cells + cnt] = td;
        ++cnt;
        break;
      }
      seg_out[r * max_cells + cnt] = te;
      ++cnt;
      double pn[3];
      exit_point(te, em, p, k, face, lo, hi, pn);
      p[0] = pn[0]; p[1] = pn[1]; p[2] = pn[2];
      wrap_slab(pb.domain, p, k);
      if (!int_coords(pb.L, p, k, X)) break;
      relocate(pb, X, stk, blockDim.x, c);
    }
  }
  n_out[r] = cnt;
}

template <class R, int NL>
__global__ void __launch_bounds__(256) k_tau(ProblemK pb, int64_t n, const double *__restrict__ orig,
                      const double *__restrict__ dir, const double *__restrict__ x_ext,
                      double *__restrict__ tau_out) {
  extern __shared__ int lds[];
  int *stk = lds + threadIdx.x;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const double p[3] = {orig[3 * r], orig[3 * r + 1], orig[3 * r + 2]};
  const double k[3] = {dir[3 * r], dir[3 * r + 1], dir[3 * r + 2]};
  double kinv[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) kinv[d] = 1.0 / k[d];
  uint32_t nc = 0;
  tau_out[r] = walk_tau<R, NL, false, false>(pb, p, k, kinv, x_ext[r], __builtin_inf(), stk, blockDim.x, &nc);
}

// ------------------------------------------------- peel-off image, adjoint
// Four waves a SIMD also in double, at 4 (one line) and 14 (more) spilled registers:
// at the three that fit without, 4e6 rays take up to 6% longer.
template <class R, int NL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) k_image_fwd(ProblemK pb, int obs, int64_t n, const double *__restrict__ orig,
                            const double *__restrict__ x_ext, const double *__restrict__ w,
                            double *__restrict__ image, unsigned long long *__restrict__ ncross) {
  extern __shared__ int lds[];
  int *stk = lds + threadIdx.x;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t nc = 0;
  if (r < n) {
    const ObsK &ob = pb.obs[obs];
    const double p[3] = {orig[3 * r], orig[3 * r + 1], orig[3 * r + 2]};
    const int pix = pixel_of(ob, p);
    if (pix >= 0) {
      const double tau = walk_tau<R, NL, sizeof(R) == 4, false>(pb, p, ob.k, ob.kinv, x_ext[r], TauCut<double>::v, stk,
                                                         blockDim.x, &nc);
      if (tau < TauCut<double>::v) unsafeAtomicAdd(image + pix, w[r] * exp(-tau));
    }
  }
  // one atomic per wave for the crossing count
  unsigned long long v = nc;
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
  if (__lane_id() == 0 && v) atomicAdd(ncross, v);
}

// Sums of a, b and c over the wave, in the lanes of rows 0, 2 and 1 (lane >> 4;
// row 3 holds 0): the three sums share their steps.  Halves are exchanged with
// v_permlane32_swap, rows with v_permlane16_swap, lanes of a row by DPP, all
// vector instructions, where butterflies through the LDS crossbar took 36
// permutes a round (1.2e8 crossings of FP32 crossing lists: 1456 -> 1309 us).
__device__ __forceinline__ double swap_add32(double x, double y) {
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)__double2loint(x), (uint32_t)__double2loint(y), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)__double2hiint(x), (uint32_t)__double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double swap_add16(double x, double y) {
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(x), (uint32_t)__double2loint(y), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(x), (uint32_t)__double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
template <int CTRL> __device__ __forceinline__ double dpp_add(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
  return x + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum3(double a, double b, double c) {
  // halves: the lower 32 lanes hold a (then c), the upper 32 b (then 0)
  double s = swap_add16(swap_add32(a, b), swap_add32(c, 0.0));   // rows: a, c, b, 0
  s = dpp_add<0x128>(s);   // row_ror 8, 4, 2, 1
  s = dpp_add<0x124>(s);
  s = dpp_add<0x122>(s);
  return dpp_add<0x121>(s);
}

// Adds each lane's (an, ak, av) to leaf `leaf` (< 0: nothing) of the
// gradients: one sum and one atomic per distinct leaf of the wave (a few
// when a wave holds rays of two sources).  Lanes that share their leaf with fewer
// than three others add their own, as do those left after four leaves; the
// groups behind a few such lanes are summed all the same (their lanes' own
// atomics on one leaf wait for each other: 1e6 FP32 rays, 37 a source, 622
// against 338 us).  Every lane of the wave must call it (cross-lane reads).
__device__ __forceinline__ void wave_leaf_add(int leaf, double an, double ak, double av, double *g_n,
                                              double *g_k, double *g_v, int lane) {
  unsigned long long m = __ballot(leaf >= 0);
  for (int round = 0; m && round < 4; ++round) {
    const int l0 = __builtin_amdgcn_readlane(leaf, __ffsll((long long)m) - 1);
    const bool mine = leaf == l0;
    const unsigned long long same = __ballot(mine);
    m &= ~same;
    // (four lanes' own atomics cost about what a sum over the wave does)
    if (__popcll(same) >= 4) {
      const double s = wave_sum3(mine ? an : 0.0, mine ? av : 0.0, mine ? ak : 0.0);
      double *const g = lane == 0 ? g_n : (lane == 16 ? g_k : g_v);
      if (lane == 0 || lane == 16 || lane == 32) unsafeAtomicAdd(g + l0, s);
      if (mine) leaf = -1;
    }
  }
  if (leaf >= 0) {
    unsafeAtomicAdd(g_n + leaf, an);
    unsafeAtomicAdd(g_k + leaf, ak);
    unsafeAtomicAdd(g_v + leaf, av);
  }
}

// Gradient terms of one crossing (segment seg of leaf record lf) of a ray
// at x_ext xr with weight g = -G_p w exp(-tau): d/dn_HI, d/dkappa_d and
// d/dv_los of g tau_c (formulas below).  In float the loop over the lines is
// kept as a loop at one line too: unrolled, the compiler fuses other products
// and the sums move by 2e-8, more than their order alone does (1e-16).
template <class R, int NL> constexpr int grad_lines() { return sizeof(R) == 4 ? MAX_LINES : NL; }

template <class R, int NL>
__device__ __forceinline__ void crossing_grad(const ProblemK &pb, const LeafRec<R> &lf, double xr, const R kr[3],
                                              double seg, double g, double inv_vth_ref, double *an, double *ak,
                                              double *av) {
  Opac<R, NL> o;
  opacity(pb, lf, xr, kr, o);
  const R b = R(pb.b_ref);
  const R den = R(1) + b * o.w;
  R sn = R(0), sv = R(0);
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    if (NL == 1 || i < pb.n_lines) {
      const LineK &ln = pb.lines[i];
      const R a = R(ln.alpha) * lf.irho;
      sn += R(ln.kfac) * voigt_h<R>(a, o.x[i]);
      const R dxdw = M<R>::div(-lf.irho * R(ln.inv_mu) * R(ln.s) * (R(1) + b * (R)xr), den * den);
      sv += R(ln.kfac) * voigt_dhdx<R>(a, o.x[i]) * dxdw;
    }
  }
  *an = g * seg * pb.box_cm * (double)lf.irho * (double)sn;
  *ak = g * seg * pb.box_cm;
  *av = g * seg * (double)lf.nl * (double)sv * inv_vth_ref;
}

// dL/dtheta_c = -G_p w exp(-tau) sum over the ray's crossings of c of
// dtau/dtheta_c, with tau_c = (nl sum_i kfac_i H_i + kd) seg:
//   dtau/dn_HI   = seg box irho sum_i kfac_i H_i
//   dtau/dkappa_d = seg box
//   dtau/dv_los  = seg nl sum_i kfac_i H'_i dx_i/dw / v_th,ref,
//   dx_i/dw = -irho inv_mu_i s_i (1 + b x_ext) / (1 + b w)^2.
template <class R, int NL, bool AXIS>
__global__ void __launch_bounds__(256) k_image_bwd(ProblemK pb, int obs, int64_t n, const double *__restrict__ orig,
                            const double *__restrict__ x_ext, const double *__restrict__ w,
                            const double *__restrict__ G, double inv_vth_ref,
                            double *__restrict__ g_n, double *__restrict__ g_k,
                            double *__restrict__ g_v, unsigned long long *__restrict__ ncross) {
  extern __shared__ int lds[];
  int *stk = lds + threadIdx.x;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = __lane_id();
  uint32_t nc = 0;
  const ObsK &ob = pb.obs[obs];
  const R kr[3] = {(R)ob.k[0], (R)ob.k[1], (R)ob.k[2]};
  bool walking = false;
  double g = 0.0, xr = 0.0;
  RayWalk<R, sizeof(R) == 4, AXIS> wk;
  uint32_t steps = 0;
  if (r < n) {
    const double p0[3] = {orig[3 * r], orig[3 * r + 1], orig[3 * r + 2]};
    const int pix = pixel_of(ob, p0);
    xr = x_ext[r];
    double tau = TauCut<double>::v;
    if (pix >= 0)
      tau = walk_tau<R, NL, sizeof(R) == 4, AXIS>(pb, p0, ob.k, ob.kinv, xr, TauCut<double>::v, stk, blockDim.x, &nc);
    g = (pix >= 0 && tau < TauCut<double>::v) ? -G[pix] * w[r] * exp(-tau) : 0.0;
    if (g != 0.0) {
      // replay the ray (same traversal as the forward pass)
      wk.p[0] = p0[0]; wk.p[1] = p0[1]; wk.p[2] = p0[2];
      walking = wk.start(pb, ob.k, stk, blockDim.x);
    }
  }
  // The wave walks its rays in step (every lane runs every iteration) so
  // that the gradient contributions of lanes in the same leaf are summed
  // across the wave first: rays from one source share their cells, and
  // one atomic per leaf replaces up to 64.  Every lane reaches the
  // shuffles below (no lane has left the loop), so their sources are live.
  while (__ballot(walking)) {
    int leaf = -1;
    double an = 0.0, ak = 0.0, av = 0.0;
    if (walking) {
      double seg;
      LeafRec<R> rec;
      walking = wk.step(pb, ob.k, ob.kinv, stk, blockDim.x, &leaf, &seg, &rec);
      crossing_grad<R, grad_lines<R, NL>()>(pb, rec, xr, kr, seg, g, inv_vth_ref, &an, &ak, &av);
      if (++steps >= MAX_CROSS) walking = false;
    }
    wave_leaf_add(leaf, an, ak, av, g_n, g_k, g_v, lane);
  }
  unsigned long long v = nc;
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
  if (lane == 0 && v) atomicAdd(ncross, v);
}

// Peel-off image of fixed rays that also records each ray's crossings (the
// tape read by k_image_bwd_tape).  The 64 rays of a wave walk in step, one
// leaf per iteration; every TAPE_CHUNK iterations the wave takes a new
// chunk (one atomic) and links it to its last one.  A wave that finds no
// chunk left goes on without recording (the host sees the count of chunks
// requested exceed the capacity and runs the pass again with more).  The
// walk and the optical depth are those of walk_tau, so the image equals the
// one k_image_fwd makes, up to the order of the additions.
template <class R, int NL, bool AXIS>
__global__ void __launch_bounds__(256) k_image_fwd_tape(ProblemK pb, int obs, int64_t n,
                                                        const double *__restrict__ orig,
                                                        const double *__restrict__ x_ext,
                                                        const double *__restrict__ w, double *__restrict__ image,
                                                        unsigned long long *__restrict__ ncross, TapeK tp) {
  extern __shared__ int lds[];
  int *stk = lds + threadIdx.x;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t wave = r >> 6;
  const int lane = __lane_id();
  const ObsK &ob = pb.obs[obs];
  const double *k = ob.k;
  const R kr[3] = {(R)k[0], (R)k[1], (R)k[2]};
  const double cut = TauCut<double>::v;
  bool walking = false;
  int pix = -1;
  double xr = 0.0, tau = 0.0;
  RayWalk<R, sizeof(R) == 4, AXIS> wk;
  uint32_t nc = 0;
  if (r < n) {
    wk.p[0] = orig[3 * r]; wk.p[1] = orig[3 * r + 1]; wk.p[2] = orig[3 * r + 2];
    pix = pixel_of(ob, wk.p);
    xr = x_ext[r];
    walking = pix >= 0 && wk.start(pb, k, stk, blockDim.x);
  }
  if (lane == 0) tp.first[wave] = -1;
  int64_t chunk = -1;   // wave-uniform
  for (uint32_t i = 0; __ballot(walking); ++i) {
    if (i % TAPE_CHUNK == 0) {
      unsigned long long q = 0;
      if (lane == 0) q = atomicAdd(tp.ctl, 1ull);
      q = __shfl(q, 0);
      const int64_t nxt = q < tp.cap ? (int64_t)q : -1;
      if (lane == 0) {
        if (i == 0) tp.first[wave] = nxt;
        else if (chunk >= 0) tp.next[chunk] = nxt;
        if (nxt >= 0) tp.next[nxt] = -1;
      }
      chunk = nxt;
    }
    if (walking) {
      int leaf;
      double seg;
      LeafRec<R> rec;
      walking = wk.step(pb, k, ob.kinv, stk, blockDim.x, &leaf, &seg, &rec);
      if (chunk >= 0) {
        const size_t e = (size_t)chunk * TAPE_ENTRIES + (size_t)(i % TAPE_CHUNK) * 64 + lane;
        tp.leaf[e] = leaf;
        ((R *)tp.seg)[e] = (R)seg;
      }
      Opac<R, NL> o;
      opacity(pb, rec, xr, kr, o);
      tau += (double)o.ktot * seg;
      ++nc;
      if (tau >= cut || nc >= MAX_CROSS) walking = false;
    }
  }
  if (r < n) {
    const double wt = (pix >= 0 && tau < cut) ? w[r] * exp(-tau) : 0.0;
    if (wt != 0.0) unsafeAtomicAdd(image + pix, wt);
    tp.count[r] = (int32_t)nc;
    tp.pix[r] = pix;
    tp.wt[r] = wt;
    tp.x[r] = xr;
  }
  unsigned long long v = nc;
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
  if (lane == 0 && v) atomicAdd(ncross, v);
}

// Adjoint of the image from the tape of the last k_image_fwd_tape pass (same
// rays, same wave of 64 rays per 64 lanes): the crossings are read back in
// the order they were walked, so no geometry and no optical depth are
// computed again.  The gradient terms and their per-leaf wave sums are
// those of k_image_bwd.
template <class R, int NL>
__global__ void __launch_bounds__(256) k_image_bwd_tape(ProblemK pb, int obs, int64_t n, TapeK tp,
                                                        const double *__restrict__ G, double inv_vth_ref,
                                                        double *__restrict__ g_n, double *__restrict__ g_k,
                                                        double *__restrict__ g_v,
                                                        unsigned long long *__restrict__ ncross) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t wave = r >> 6;
  const int lane = __lane_id();
  const double *k = pb.obs[obs].k;
  const R kr[3] = {(R)k[0], (R)k[1], (R)k[2]};
  double g = 0.0, xr = 0.0;
  int cnt = 0;
  if (r < n) {
    const double wt = tp.wt[r];
    if (wt != 0.0) {
      g = -G[tp.pix[r]] * wt;
      if (g != 0.0) {
        cnt = tp.count[r];
        xr = tp.x[r];
      }
    }
  }
  // wave iterations needed: the longest crossing list among lanes with a
  // gradient (every lane's list starts at the wave's first iteration)
  int m = cnt;
  for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off));
  int64_t chunk = m > 0 ? tp.first[wave] : -1;
  for (int i = 0; i < m; ++i) {
    if (i > 0 && i % TAPE_CHUNK == 0) chunk = tp.next[chunk];
    if (chunk < 0) break;   // an incomplete tape (the host never passes one)
    int leaf = -1;
    double an = 0.0, ak = 0.0, av = 0.0;
    if (i < cnt) {
      const size_t e = (size_t)chunk * TAPE_ENTRIES + (size_t)(i % TAPE_CHUNK) * 64 + lane;
      leaf = tp.leaf[e];
      const double seg = (double)((const R *)tp.seg)[e];
      const LeafRec<R> lf = load_leaf<R>(pb.leaves, leaf);
      crossing_grad<R, grad_lines<R, NL>()>(pb, lf, xr, kr, seg, g, inv_vth_ref, &an, &ak, &av);
    }
    wave_leaf_add(leaf, an, ak, av, g_n, g_k, g_v, lane);
  }
  unsigned long long v = (unsigned long long)cnt;
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
  if (lane == 0 && v) atomicAdd(ncross, v);
}

// ----------------------------------------------------- gas and sources in
// Gas fields as given (float or double; v is [3n]) checked and copied into
// the raw per-leaf array raw[8n] = {n_HI, T, vx, vy, vz, kappa_d, 0, 0} in
// double.  bad[0] receives the smallest leaf with a non-finite or negative
// value (or T <= 0), bad[1] the smallest with a velocity component of at
// least 0.1 c; both start at ~0 (set by the caller).
template <class T>
__global__ void k_stage_gas(int64_t n, const T *__restrict__ nh, const T *__restrict__ tk,
                            const T *__restrict__ v, const T *__restrict__ kd, double *__restrict__ raw,
                            unsigned long long *__restrict__ bad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double a = (double)nh[i], t = (double)tk[i], k = (double)kd[i];
  const double vx = (double)v[3 * i], vy = (double)v[3 * i + 1], vz = (double)v[3 * i + 2];
  const bool ok = isfinite(a) && a >= 0.0 && isfinite(t) && t > 0.0 && isfinite(k) && k >= 0.0 && isfinite(vx) &&
                  isfinite(vy) && isfinite(vz);
  const double vmax = 0.1 * 2.99792458e10;
  if (!ok) atomicMin(bad, (unsigned long long)i);
  else if (fabs(vx) >= vmax || fabs(vy) >= vmax || fabs(vz) >= vmax) atomicMin(bad + 1, (unsigned long long)i);
  double *r = raw + 8 * i;
  r[0] = a; r[1] = t; r[2] = vx; r[3] = vy; r[4] = vz; r[5] = k; r[6] = 0.0; r[7] = 0.0;
}

// Leaf records (see rmc_device.h) from the raw gas: nl = n_HI box irho,
// irho = sqrt(T_ref / T), kd = kappa_d box, u = v / v_th,ref, and the
// domain-border flag of the leaf (level lv, integer coordinates ijk at its
// level): box -- touches a face of the cube; slab -- not strictly inside
// the slab; sphere -- some corner outside R (1 - 1e-9).  Plain IEEE double
// arithmetic, uncontracted, so the records are exact functions of the
// inputs; the float path rounds them once.
#pragma clang fp contract(off)
template <class R>
__global__ void k_leaf_records(int64_t n, const double *__restrict__ raw, const int8_t *__restrict__ lv,
                               const int32_t *__restrict__ ijk, double T_ref, double vth_ref, double box,
                               int domain, double d0, double d1, double d2, double d3, R *__restrict__ leaves) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double *g = raw + 8 * i;
  const double irho = sqrt(T_ref / g[1]);
  const int l = lv[i];
  const double h = ldexp(1.0, -l);
  double lo[3], hi[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = (double)ijk[3 * i + d] * h;
    hi[d] = (double)(ijk[3 * i + d] + 1) * h;
  }
  bool border;
  if (domain == DOM_BOX) {
    border = lo[0] <= 0.0 || hi[0] >= 1.0 || lo[1] <= 0.0 || hi[1] >= 1.0 || lo[2] <= 0.0 || hi[2] >= 1.0;
  } else if (domain == DOM_SLAB_Z) {
    border = !(lo[2] > d0 - d1 && hi[2] < d0 + d1);
  } else {
    const double Rr = d3 * (1.0 - 1e-9);
    const double c[3] = {d0, d1, d2};
    double far2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double a = fabs(lo[d] - c[d]), b = fabs(hi[d] - c[d]);
      const double m = a > b ? a : b;
      far2 += m * m;
    }
    border = !(far2 < Rr * Rr);
  }
  const double rec[8] = {g[0] * box * irho, irho, g[5] * box, g[2] / vth_ref, g[3] / vth_ref, g[4] / vth_ref,
                         border ? 1.0 : 0.0, log10(irho)};
  R *o = leaves + (size_t)i * LEAF_STRIDE;
#pragma unroll
  for (int q = 0; q < 8; ++q) o[q] = (R)rec[q];
}

// Device-resident sources checked as the host path checks them: positions
// in [0,1], finite x, unit directions (|k|^2 within 1e-6 of 1).  bad[0]
// receives the smallest failing source.
__global__ void k_check_sources(int64_t n, const double *__restrict__ pos, const double *__restrict__ dir,
                                const double *__restrict__ x, unsigned long long *__restrict__ bad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  bool ok = isfinite(x[i]);
#pragma unroll
  for (int d = 0; d < 3; ++d) ok = ok && pos[3 * i + d] >= 0.0 && pos[3 * i + d] <= 1.0;
  if (dir) {
    const double nn = dir[3 * i] * dir[3 * i] + dir[3 * i + 1] * dir[3 * i + 1] + dir[3 * i + 2] * dir[3 * i + 2];
    ok = ok && fabs(nn - 1.0) < 1e-6;
  }
  if (!ok) atomicMin(bad, (unsigned long long)i);
}

// Gradient with respect to the cell velocity vector from the one with
// respect to v_los = k_obs . v (chain rule): g_v[3i + d] = g_vlos[i] k_d.
__global__ void k_vlos_to_v(int64_t n, const double *__restrict__ g_vlos, double k0, double k1, double k2,
                            double *__restrict__ g_v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double g = g_vlos[i];
  g_v[3 * i] = g * k0;
  g_v[3 * i + 1] = g * k1;
  g_v[3 * i + 2] = g * k2;
}
#pragma clang fp contract(fast)

// --------------------------------------------------------------- helpers
// The bin of packet i, or -1 (not escaped, or outside the range).
__device__ __forceinline__ int hist_bin(int32_t status, double x, int nbins, double x_min, double span) {
  const double fb = (x - x_min) / span * nbins;
  if (status != ST_ESCAPED || !(fb >= 0.0 && fb < nbins)) return -1;
  const int b = (int)floor(fb);
  return b < nbins ? b : -1;
}

// Spectrum of escaped packets.  Most of them share a few hundred bins, and
// atomics on one address wait for each other: each block counts its packets in
// LDS and adds its non-zero bins.  2e6 packets in 700 bins: 28 us, with one atomic
// a packet 980 us.
__global__ void __launch_bounds__(256) k_hist(int64_t n, const int32_t *__restrict__ status,
                                              const double *__restrict__ x, int nbins, double x_min, double span,
                                              unsigned long long *__restrict__ h) {
  extern __shared__ int lds[];
  unsigned *const cnt = (unsigned *)lds;
  for (int b = threadIdx.x; b < nbins; b += blockDim.x) cnt[b] = 0u;
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int b = hist_bin(status[i], x[i], nbins, x_min, span);
    if (b >= 0) atomicAdd(cnt + b, 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbins; b += blockDim.x)
    if (cnt[b]) atomicAdd(h + b, (unsigned long long)cnt[b]);
}

// The same with an atomic a packet, for more bins than a block's LDS holds.
__global__ void k_hist_wide(int64_t n, const int32_t *__restrict__ status, const double *__restrict__ x, int nbins,
                            double x_min, double span, unsigned long long *__restrict__ h) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int b = hist_bin(status[i], x[i], nbins, x_min, span);
  if (b >= 0) atomicAdd(h + b, 1ull);
}

// Zero the counters of every problem of a launch, the work queue and its
// waves' reserves (a kernel rather than a memset so that it can sit in a captured graph).
__global__ void k_batch_reset(const ProblemK *__restrict__ probs, int n, unsigned long long *next, int waves) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n * N_STATS) probs[i / N_STATS].stats[i % N_STATS] = 0ull;
  if (i < RESERVE_OFFSET + 2 * waves) next[i] = 0ull;
}

__global__ void k_fill_u64(unsigned long long *p, int64_t n, unsigned long long v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_u64_to_f64(const unsigned long long *a, double *b, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (double)a[i];
}

__global__ void k_f32_to_f64(const float *a, double *b, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (double)a[i];
}

__global__ void k_f64_to_f32(const double *a, float *b, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (float)a[i];
}

// ------------------------------------------ fixed scratch (no allocation)
// Histogram counts of rmc_get_spectrum_noalloc: a file-scope device array
// of NOALLOC_MAX_BINS counters (each device the library runs on holds its
// own copy until the process ends).  Host code never uses the array's name
// as an address: scratch_address() asks the runtime for the current
// device's copy once and keeps it.
static __device__ __align__(256) unsigned long long scratch[NOALLOC_MAX_BINS];

hipError_t scratch_address(int device, unsigned long long **out) {
  static std::mutex mu;
  static unsigned long long *addr[256] = {};
  if (device < 0 || device >= 256) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[device] = (unsigned long long *)p;
  }
  *out = addr[device];
  return hipSuccess;
}

// ------------------------------------------------------------- launchers
static inline unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

using TransportFn = void (*)(const ProblemK *, const int64_t *, int, unsigned long long *, int, int, SlotState *,
                            int, unsigned long long *);

// The one-round-per-pass form (regroup) is built for the deferred
// peel-off kernels only (the default).
template <class R, int NL>
static TransportFn transport_fn(bool batch, bool defer, bool regroup) {
  if (batch) {
    if (!defer) return k_transport<R, true, false, NL>;
    return regroup ? k_transport<R, true, true, NL, true> : k_transport<R, true, true, NL>;
  }
  if (!defer) return k_transport<R, false, false, NL>;
  return regroup ? k_transport<R, false, true, NL, true> : k_transport<R, false, true, NL>;
}

static TransportFn transport_fn(bool fp32, bool batch, bool defer, int nl, bool regroup) {
  if (fp32)
    return nl == 1   ? transport_fn<float, 1>(batch, defer, regroup)
           : nl == 2 ? transport_fn<float, 2>(batch, defer, regroup)
                     : transport_fn<float, MAX_LINES>(batch, defer, regroup);
  return nl == 1   ? transport_fn<double, 1>(batch, defer, regroup)
         : nl == 2 ? transport_fn<double, 2>(batch, defer, regroup)
                   : transport_fn<double, MAX_LINES>(batch, defer, regroup);
}

static size_t transport_lds(int stack_levels, int block) {
  return ((size_t)2 * stack_levels * block + WAVE_WORDS * (block / 64)) * sizeof(int);
}

hipError_t launch_transport(bool fp32, bool batch, bool defer, int nl, bool regroup, const ProblemK *d_probs,
                            const int64_t *d_starts, int n_probs, unsigned long long *d_next, int refill_min,
                            int stack_levels, int grid, int block, void *slots, int budget,
                            unsigned long long *slice, hipStream_t st) {
  hipLaunchKernelGGL(transport_fn(fp32, batch, defer, nl, regroup), dim3(grid), dim3(block),
                     transport_lds(stack_levels, block), st,
                     d_probs, d_starts, n_probs, d_next, refill_min, stack_levels, (SlotState *)slots, budget, slice);
  return hipGetLastError();
}

template <class R>
static void launch_walkers_as(bool batch, int nl, const ProblemK *d_probs, int region0, int levels,
                              SlotState *slots, int lp, int waves, int budget, unsigned long long *slice,
                              hipStream_t st) {
  const auto fn = batch ? (nl == 1 ? k_walkers<R, true, 1> : nl == 2 ? k_walkers<R, true, 2> : k_walkers<R, true, MAX_LINES>)
                        : (nl == 1   ? k_walkers<R, false, 1>
                           : nl == 2 ? k_walkers<R, false, 2>
                                     : k_walkers<R, false, MAX_LINES>);
  hipLaunchKernelGGL(fn, dim3(waves), dim3(64), (size_t)levels * 64 * sizeof(int), st, d_probs, region0, slots, lp,
                     budget, slice);
}

hipError_t launch_walkers(bool fp32, bool batch, int nl, const ProblemK *d_probs, int region0, int stack_levels,
                          void *slots, int lp, int waves, int budget, unsigned long long *slice, hipStream_t st) {
  SlotState *s = (SlotState *)slots;
  if (fp32) launch_walkers_as<float>(batch, nl, d_probs, region0, stack_levels, s, lp, waves, budget, slice, st);
  else launch_walkers_as<double>(batch, nl, d_probs, region0, stack_levels, s, lp, waves, budget, slice, st);
  return hipGetLastError();
}

hipError_t launch_group_slots(const void *src, int64_t n, void *dst, int64_t n_dst, int n_probs, int lp, uint32_t *work,
                              unsigned long long *n_live, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_group_count, dim3(blocks_for(n, 256)), dim3(256), 0, st, (const SlotState *)src, n, work);
  hipLaunchKernelGGL(k_group_offsets, dim3(1), dim3(1024), 0, st, work, n_probs, lp, n_live);
  hipLaunchKernelGGL(k_group_slots, dim3(blocks_for(n, 256)), dim3(256), 0, st, (const SlotState *)src, n,
                     (SlotState *)dst, n_dst, work);
  return hipGetLastError();
}

using DrainFn = void (*)(const ProblemK *, PeelQueue *, unsigned long long *);

template <class R, int NL>
static DrainFn drain_fn(bool batch, bool one) {
  return batch ? k_peel_drain<R, true, false, NL> : one ? k_peel_drain<R, false, true, NL> : k_peel_drain<R, false, false, NL>;
}

static DrainFn drain_fn(bool fp32, bool batch, bool one, int nl) {
  if (nl == 1) return fp32 ? drain_fn<float, 1>(batch, one) : drain_fn<double, 1>(batch, one);
  if (nl == 2) return fp32 ? drain_fn<float, 2>(batch, one) : drain_fn<double, 2>(batch, one);
  return fp32 ? drain_fn<float, MAX_LINES>(batch, one) : drain_fn<double, MAX_LINES>(batch, one);
}

hipError_t launch_peel_drain(bool fp32, bool batch, bool one, int nl, const ProblemK *d_probs, void *pq,
                             int n_regions, int stack_levels, int grid, unsigned long long *slice, hipStream_t st) {
  const int b = 256;
  const size_t lds = (size_t)stack_levels * b * sizeof(int);
  PeelQueue *q = (PeelQueue *)pq;
  hipLaunchKernelGGL(k_peel_scan, dim3(1), dim3(1024), 0, st, q, n_regions, slice);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(drain_fn(fp32, batch, one, nl), dim3(grid), dim3(b), lds, st, d_probs, q, slice);
  return hipGetLastError();
}

int peel_drain_blocks_per_cu(bool fp32, bool batch, bool one, int nl, int stack_levels) {
  const size_t lds = (size_t)stack_levels * 256 * sizeof(int);
  int nb = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, drain_fn(fp32, batch, one, nl), 256, lds);
  return (e == hipSuccess && nb > 0) ? nb : 1;
}

size_t peel_job_bytes(bool fp32) { return fp32 ? sizeof(PeelJob<float>) : sizeof(PeelJob<double>); }
size_t peel_queue_bytes() { return sizeof(PeelQueue); }

size_t slot_bytes() { return sizeof(SlotState); }

int transport_blocks_per_cu(bool fp32, bool batch, bool defer, int nl, bool regroup, int block,
                            int stack_levels) {
  int nb = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb,
                                                                    transport_fn(fp32, batch, defer, nl, regroup),
                                                                    block,
                                                                    transport_lds(stack_levels, block));
  return (e == hipSuccess && nb > 0) ? nb : 1;
}

hipError_t launch_clear_slots(void *slots, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_clear_slots, dim3(blocks_for(n, 256)), dim3(256), 0, st, (SlotState *)slots, n);
  return hipGetLastError();
}

hipError_t launch_compact_slots(const void *src, int64_t n, void *dst, unsigned long long *n_live,
                                hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_compact_slots, dim3(blocks_for(n, 256)), dim3(256), 0, st, (const SlotState *)src, n,
                     (SlotState *)dst, n_live);
  return hipGetLastError();
}

hipError_t launch_count_live(const void *slots, int64_t n, unsigned long long *out, hipStream_t st) {
  hipLaunchKernelGGL(k_count_live, dim3(blocks_for(n, 256)), dim3(256), 0, st, (const SlotState *)slots, n, out);
  return hipGetLastError();
}

hipError_t launch_trace(const ProblemK &pb, int64_t n, const double *orig, const double *dir,
                        int max_cells, int32_t *leaf, double *seg, int32_t *cnt, hipStream_t st) {
  const int b = 256;
  const size_t lds = (size_t)(pb.L > 0 ? pb.L : 1) * b * sizeof(int);
  hipLaunchKernelGGL(k_trace, dim3(blocks_for(n, b)), dim3(b), lds, st, pb, n, orig, dir, max_cells, leaf,
                     seg, cnt);
  return hipGetLastError();
}

// Threads per block of the ray kernels: one wave where blocks of four waves would
// not give each CU one.  A ray is a serial chain, and single waves
// spread over the CUs.  FP64 optical depths with their copies, blocks of 256 ->
// of 64 threads: 5000 rays 400 -> 329 us, 20001 rays 436 -> 403; from 65536 rays
// (525 and 524) to 1e6 both take the same within 2%.
static int ray_block(int64_t n) {
  constexpr int64_t cus = 256;   // of the one device this library is compiled for
  return n < cus * 256 ? 64 : 256;
}

// Whether an observer's rays move along one axis only: then the double tape and
// both backward kernels branch round the others (AXIS of RayWalk), 3-5% faster
// there from 3e5 rays on.  The other ray kernels are no slower without, and rays
// that move along two axes are faster without in all of them.
static bool along_axis(const ObsK &ob) {
  return (ob.k[0] != 0.0) + (ob.k[1] != 0.0) + (ob.k[2] != 0.0) == 1;
}

hipError_t launch_tau(bool fp32, const ProblemK &pb, int64_t n, const double *orig, const double *dir,
                      const double *x, double *tau, hipStream_t st) {
  const int b = ray_block(n);
  const size_t lds = (size_t)(pb.L > 0 ? pb.L : 1) * b * sizeof(int);
  const auto fn = fp32 ? (pb.n_lines == 1 ? k_tau<float, 1> : k_tau<float, MAX_LINES>)
                       : (pb.n_lines == 1 ? k_tau<double, 1> : k_tau<double, MAX_LINES>);
  hipLaunchKernelGGL(fn, dim3(blocks_for(n, b)), dim3(b), lds, st, pb, n, orig, dir, x, tau);
  return hipGetLastError();
}

hipError_t launch_image_fwd(bool fp32, const ProblemK &pb, int obs, int64_t n, const double *orig,
                            const double *x, const double *w, double *image, unsigned long long *ncross,
                            hipStream_t st) {
  const int b = ray_block(n);
  const size_t lds = (size_t)(pb.L > 0 ? pb.L : 1) * b * sizeof(int);
  const auto fn = fp32 ? (pb.n_lines == 1 ? k_image_fwd<float, 1> : k_image_fwd<float, MAX_LINES>)
                       : (pb.n_lines == 1 ? k_image_fwd<double, 1> : k_image_fwd<double, MAX_LINES>);
  hipLaunchKernelGGL(fn, dim3(blocks_for(n, b)), dim3(b), lds, st, pb, obs, n, orig, x, w, image, ncross);
  return hipGetLastError();
}

hipError_t launch_image_bwd(bool fp32, const ProblemK &pb, int obs, int64_t n, const double *orig,
                            const double *x, const double *w, const double *G, double inv_vth_ref,
                            double *gn, double *gk, double *gv, unsigned long long *ncross, hipStream_t st) {
  const int b = ray_block(n);
  const size_t lds = (size_t)(pb.L > 0 ? pb.L : 1) * b * sizeof(int);
  const bool axis = along_axis(pb.obs[obs]), one = pb.n_lines == 1;
  const auto fn = fp32 ? (axis ? (one ? k_image_bwd<float, 1, true> : k_image_bwd<float, MAX_LINES, true>)
                               : (one ? k_image_bwd<float, 1, false> : k_image_bwd<float, MAX_LINES, false>))
                       : (axis ? (one ? k_image_bwd<double, 1, true> : k_image_bwd<double, MAX_LINES, true>)
                               : (one ? k_image_bwd<double, 1, false> : k_image_bwd<double, MAX_LINES, false>));
  hipLaunchKernelGGL(fn, dim3(blocks_for(n, b)), dim3(b), lds, st, pb, obs, n, orig, x, w, G, inv_vth_ref, gn, gk, gv, ncross);
  return hipGetLastError();
}

int64_t tape_waves(int64_t n) { return (int64_t)blocks_for(n, 256) * 4; }

hipError_t launch_image_fwd_tape(bool fp32, const ProblemK &pb, int obs, int64_t n, const double *orig,
                                 const double *x, const double *w, double *image, unsigned long long *ncross,
                                 const TapeK &tp, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int b = 256;
  const size_t lds = (size_t)(pb.L > 0 ? pb.L : 1) * b * sizeof(int);
  const bool axis = along_axis(pb.obs[obs]), one = pb.n_lines == 1;
  const auto fn = fp32 ? (one ? k_image_fwd_tape<float, 1, false> : k_image_fwd_tape<float, MAX_LINES, false>)
                       : (axis ? (one ? k_image_fwd_tape<double, 1, true> : k_image_fwd_tape<double, MAX_LINES, true>)
                               : (one ? k_image_fwd_tape<double, 1, false> : k_image_fwd_tape<double, MAX_LINES, false>));
  hipLaunchKernelGGL(fn, dim3(blocks_for(n, b)), dim3(b), lds, st, pb, obs, n, orig, x, w, image, ncross, tp);
  return hipGetLastError();
}

hipError_t launch_image_bwd_tape(bool fp32, const ProblemK &pb, int obs, int64_t n, const TapeK &tp,
                                 const double *G, double inv_vth_ref, double *gn, double *gk, double *gv,
                                 unsigned long long *ncross, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int b = 256;
  const auto fn = fp32 ? (pb.n_lines == 1 ? k_image_bwd_tape<float, 1> : k_image_bwd_tape<float, MAX_LINES>)
                       : (pb.n_lines == 1 ? k_image_bwd_tape<double, 1> : k_image_bwd_tape<double, MAX_LINES>);
  hipLaunchKernelGGL(fn, dim3(blocks_for(n, b)), dim3(b), 0, st, pb, obs, n, tp, G, inv_vth_ref, gn, gk, gv, ncross);
  return hipGetLastError();
}

hipError_t launch_stage_gas(bool f32_in, int64_t n, const void *nh, const void *tk, const void *v, const void *kd,
                           double *raw, unsigned long long *bad, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (f32_in)
    hipLaunchKernelGGL(k_stage_gas<float>, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, (const float *)nh,
                       (const float *)tk, (const float *)v, (const float *)kd, raw, bad);
  else
    hipLaunchKernelGGL(k_stage_gas<double>, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, (const double *)nh,
                       (const double *)tk, (const double *)v, (const double *)kd, raw, bad);
  return hipGetLastError();
}

hipError_t launch_leaf_records(bool fp32, int64_t n, const double *raw, const int8_t *lv, const int32_t *ijk,
                               double T_ref, double vth_ref, double box, int domain, const double dom[4],
                               void *leaves, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (fp32)
    hipLaunchKernelGGL(k_leaf_records<float>, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, raw, lv, ijk, T_ref,
                       vth_ref, box, domain, dom[0], dom[1], dom[2], dom[3], (float *)leaves);
  else
    hipLaunchKernelGGL(k_leaf_records<double>, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, raw, lv, ijk, T_ref,
                       vth_ref, box, domain, dom[0], dom[1], dom[2], dom[3], (double *)leaves);
  return hipGetLastError();
}

hipError_t launch_check_sources(int64_t n, const double *pos, const double *dir, const double *x,
                                unsigned long long *bad, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_check_sources, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, pos, dir, x, bad);
  return hipGetLastError();
}

hipError_t launch_vlos_to_v(int64_t n, const double *g_vlos, const double k[3], double *g_v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_vlos_to_v, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, g_vlos, k[0], k[1], k[2], g_v);
  return hipGetLastError();
}

// Bins of a block's LDS counters (32 KB: four blocks a CU), and blocks of a
// large launch: four a CU.
constexpr int HIST_LDS_BINS = 8192;
constexpr int HIST_BLOCKS = 1024;

hipError_t launch_hist(int64_t n, const int32_t *status, const double *x, int nbins, double x_min, double span,
                       unsigned long long *h, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  // a block's 32-bit counts hold its share of the packets (n < 2^31)
  if (nbins <= HIST_LDS_BINS && n < ((int64_t)1 << 31)) {
    const int blocks = n < 256 * HIST_BLOCKS ? blocks_for(n, 256) : HIST_BLOCKS;
    hipLaunchKernelGGL(k_hist, dim3(blocks), dim3(256), (size_t)nbins * sizeof(unsigned), st, n, status, x, nbins,
                       x_min, span, h);
  } else {
    hipLaunchKernelGGL(k_hist_wide, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, status, x, nbins, x_min, span, h);
  }
  return hipGetLastError();
}

hipError_t launch_batch_reset(const ProblemK *d_probs, int n, unsigned long long *d_next, int waves,
                              hipStream_t st) {
  const int64_t m = (int64_t)n * N_STATS, w = RESERVE_OFFSET + 2 * (int64_t)waves;
  hipLaunchKernelGGL(k_batch_reset, dim3(blocks_for(m > w ? m : w, 256)), dim3(256), 0, st, d_probs, n, d_next, waves);
  return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u64, dim3(blocks_for(n, 256)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

hipError_t launch_u64_to_f64(const unsigned long long *a, double *b, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_u64_to_f64, dim3(blocks_for(n, 256)), dim3(256), 0, st, a, b, n);
  return hipGetLastError();
}

hipError_t launch_f32_to_f64(const float *a, double *b, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_f32_to_f64, dim3(blocks_for(n, 256)), dim3(256), 0, st, a, b, n);
  return hipGetLastError();
}

hipError_t launch_f64_to_f32(const double *a, float *b, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_f64_to_f32, dim3(blocks_for(n, 256)), dim3(256), 0, st, a, b, n);
  return hipGetLastError();
}

}  // namespace rmc
