// Persistent tracking kernel: one lane per particle, all turns and all
// elements of the ring in one launch, state in registers.
//
// Per element (wave-uniform walk of the lattice index sequence):
//   drift            exact flow, no spin
//   sector bend      exact steps of ds between slice edges (§3.1)
//   quadrupole       DKD or MK slices (§3.4, §3.3)
//   thin multipole   half kick, rotation by the integrated Ω, half kick
//   snake            fixed rotation
// Thick elements with spin evaluate Ω at the N + 1 slice edges (§4.3) and
// fold each edge into the running product of every Romberg level that keeps
// it, so no Ω record ever leaves the registers.  The tableau and the
// normalisation follow at the element exit, and the element quaternion is
// composed into the turn quaternion, which rotates the spin once per turn.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "fp64_maps.h"
#include "mixed_spin.h"
#include "track_kernels.h"

namespace st {

namespace {

constexpr int kBlock = 256;

typedef const DevElem __attribute__((address_space(4))) ConstElem;
typedef const Record __attribute__((address_space(4))) ConstRecord;
typedef const uint32_t __attribute__((address_space(4))) ConstSeq;

// Member-wise copy of one element record out of the constant address space
// (uniform address: scalar loads).
__device__ __forceinline__ DevElem load_elem(const ConstElem* p) {
  DevElem d;
  d.kind = p->kind;
  d.orbit = p->orbit;
  d.nsl = p->nsl;
  d.K = p->K;
  d.flags = p->flags;
  d.place = p->place;
  d.hw_end = p->hw_end;
  d.hw_in = p->hw_in;
  d.hw2_end = p->hw2_end;
  d.hw2_in = p->hw2_in;
  #pragma unroll
  for (int i = 0; i < kElemWords; ++i) d.v[i] = p->v[i];
  return d;
}

__device__ __forceinline__ Record load_record(const ConstRecord* p) {
  Record r;
  r.op = p->op;
  r.flags = p->flags;
  r.count = p->count;
  r.elem = p->elem;
  r.tail = p->tail;
#pragma unroll
  for (int i = 0; i < kHotWords; ++i) r.v[i] = p->v[i];
  return r;
}

// Waves per SIMD the register allocation aims at: two, for every variant.
// The plain double kernel fits in 238 VGPRs with no scratch at two waves (the
// mixed one in 232 with 40 B a lane); at three waves (168 VGPRs) an earlier form
// ran at the same speed, but spilled 70 VGPRs at the element entrances, and with
// 2^20 lanes those spill slots (228 B each) were written back to memory, about
// 500 GB per 100-turn launch.
#ifndef ST_WAVES_PER_EU
#define ST_WAVES_PER_EU 2
#endif
#ifndef ST_WAVES_PER_EU_WIDE
#define ST_WAVES_PER_EU_WIDE 2
#endif
#ifndef ST_WAVES_PER_EU_ORBIT
#define ST_WAVES_PER_EU_ORBIT 4
#endif

// Romberg spin integration through one thick element, fused with its orbit
// slices (KIND: 0 sector bend, 1 MK quadrupole focusing in x, 3 MK
// quadrupole focusing in y, 2 DKD quadrupole, 4 drift-kick (TEAPOT) sector
// bend).  In the MIXED kernel,
// elements flagged F_SPIN32 use single-precision edge quaternions and
// compensated single-precision level products.  Returns the normalised
// element quaternion.
// One second-order quadrupole step over the length of q: matrix-kick-matrix
// (KIND 1 focusing in x, 3 focusing in y) or drift-kick-drift (KIND 2).
template <int KIND, bool CLOSED>
__device__ __forceinline__ void quad_step2(const QuadParams& q, const MKConst& mc, double& X,
                                           double& Px, double& Y, double& Py, double& T,
                                           const Particle& p, const TrackArgs& a, bool& beyond) {
  if (KIND == 1) {
    mk_linear(mc, X, Px, Y, Py, T, p);
    mk_nonlinear<CLOSED>(q.ds, X, Px, Y, Py, T, p, beyond);
    mk_linear(mc, X, Px, Y, Py, T, p);
  } else if (KIND == 3) {
    mk_linear(mc, Y, Py, X, Px, T, p);
    mk_nonlinear<CLOSED>(q.ds, X, Px, Y, Py, T, p, beyond);
    mk_linear(mc, Y, Py, X, Px, T, p);
  } else {
    drift_part<CLOSED>(q.hds, X, Px, Y, Py, T, p, a.inv_beta0, beyond);
    Px = fma(-q.k1ds, X, Px);
    Py = fma(q.k1ds, Y, Py);
    drift_part<CLOSED>(q.hds, X, Px, Y, Py, T, p, a.inv_beta0, beyond);
  }
}

// Fourth-order quadrupole slice (orbit methods DKD4, MK4): the second-order
// step over x1 ds, x0 ds and x1 ds (2 x1 + x0 = 1, 2 x1^3 + x0^3 = 0).  m1 and
// m0 are the MK constants of the two step lengths.
template <int KIND, bool CLOSED>
__device__ __forceinline__ void quad_slice4(const Quad4Params& q4, const MKConst& m1,
                                            const MKConst& m0, double& X, double& Px, double& Y,
                                            double& Py, double& T, const Particle& p,
                                            const TrackArgs& a, bool& beyond) {
  quad_step2<KIND, CLOSED>(q4.s1, m1, X, Px, Y, Py, T, p, a, beyond);
  quad_step2<KIND, CLOSED>(q4.s0, m0, X, Px, Y, Py, T, p, a, beyond);
  quad_step2<KIND, CLOSED>(q4.s1, m1, X, Px, Y, Py, T, p, a, beyond);
}

// Matrix-kick constants of the last quadrupole a lane crossed, kept in the
// block's LDS (one column per lane).  They depend only on the particle's P
// and on the element's |k1| and slice length, so quadrupoles that share
// those (in a FODO ring the focusing and defocusing ones usually do) reuse
// them instead of re-evaluating the series.  The key is element data, the
// same for every lane of a wave.
constexpr int kMKWords = sizeof(MKLin) / sizeof(double);
struct MKCache {
  double* slot;            // the lane's word of the first row
  int stride;              // between rows
  double k1abs, hds;       // key of the stored constants (NaN: none yet)
};

__device__ __forceinline__ MKLin mk_cached(const QuadParams& q, const Particle& p, MKCache* c) {
  MKLin m;
  double* w = reinterpret_cast<double*>(&m);
  const double ka = fabs(q.k1);
  if (c && ka == c->k1abs && q.hds == c->hds) {
#pragma unroll
    for (int i = 0; i < kMKWords; ++i) w[i] = c->slot[i * c->stride];
    return m;
  }
  m = mk_lin(q, p);
  if (c) {
#pragma unroll
    for (int i = 0; i < kMKWords; ++i) c->slot[i * c->stride] = w[i];
    c->k1abs = ka;
    c->hds = q.hds;
  }
  return m;
}

// One matrix-kick slice, orbit only (KIND 1 focusing in x, 3 in y); tk
// collects the kick's flight time (mk_flight).
template <int KIND, bool CLOSED>
__device__ __forceinline__ void mk_slice(const QuadParams& q, const MKLin& m, double& X, double& Px,
                                         double& Y, double& Py, double& tk, const Particle& p,
                                         bool& beyond) {
  if (KIND == 1) mk_move(m, X, Px, Y, Py);
  else           mk_move(m, Y, Py, X, Px);
  mk_kick<CLOSED>(q.ds, X, Px, Y, Py, tk, p, beyond);
  if (KIND == 1) mk_move(m, X, Px, Y, Py);
  else           mk_move(m, Y, Py, X, Px);
}

// Y4: quadrupoles with the fourth-order slice (extended kernels only).
// PEEL: the entrance edge is folded outside the slice loop, where the level
// products are set instead of multiplied into the identity (the extended
// kernels keep one copy of the edge code, which holds their registers down).
template <int NT, int KIND, bool MIXED, bool Y4 = false, bool PEEL = true>
__device__ __forceinline__ Quat thick_element(const DevElem& el, double& X, double& Px, double& Y,
                                              double& Py, double& T, const Particle& p,
                                              const TrackArgs& a, MKCache* mkc = nullptr) {
  static_assert(kMaxRows == 4, "the level products below are written out for four rows");
  const bool all_closed = KIND == 4 && el.tp.closed != 0.0;
  const int N = el.nsl;
  const int K = el.K;
  const double ds = KIND == 0 ? el.b.ds : (KIND == 4 ? el.tp.ds : el.q.ds);
  // MIXED: this element's edges are built and multiplied in single
  // precision (the caller picks this instantiation for flagged elements)
  constexpr bool spin32 = MIXED;
  // running products of the Romberg levels: level m keeps every 2^m-th edge
  Quat Q0 = qident(), Q1 = qident(), Q2 = qident(), Q3 = qident();
  QuatC C0 = qc_ident(), C1 = qc_ident(), C2 = qc_ident(), C3 = qc_ident();

  // bend invariants of this particle: Py and Pt do not change in a bend
  double Pa2 = p.P2() - Py * Py;
  constexpr bool MK = (KIND == 1 || KIND == 3) && !Y4;
  MKConst mc, mc0;
  MKLin ml;
  double kP = 0.0, esum = 0.0, tk = 0.0, xp_in = 0.0;   // flight time (mk_flight)
  if constexpr (MK) {
    ml = mk_cached(el.q, p, mkc);
    kP = fabs(el.q.k1) * p.P();
    xp_in = fma(X, Px, Y * Py);
  } else if (KIND == 1 || KIND == 3) {
    mc = mk_const(el.q4.s1, p);
    mc0 = mk_const(el.q4.s0, p);
  }
  auto invariant = [&](double w) {
    const double pp = fma(Px, Px, Py * Py);
    esum = fma(w, KIND == 1 ? mk_invariant(kP, pp, X, Y) : mk_invariant(kP, pp, Y, X), esum);
  };
  if constexpr (MK) invariant(0.5);

  // Ps and 1/Ps at the entrance edge (outside bends 1/Ps only enters Ω)
  double ps2 = fma(-Px, Px, Pa2);
  double r = KIND == 0 ? rsqrt_nr(ps2) : rsqrt_omega(ps2);
  double W = ps2 * r;
  double invPa2 = 0.0, wme = 0.0;
  // entrance Px and Ps of a bend: Y and T follow once from the two ends
  const double Px_in = Px, W_in = W;
  if (KIND == 0) {
    invPa2 = rcp_nr(Pa2);
    // W - η = (W² - η²)/(W + η) with W² - η² = (1 - η²) + (P² - 1) - Py² - Px²
    wme = (el.b.one_m_eta2 + ((p.c3 - Py * Py) - Px * Px)) * rcp_nr(W + el.b.eta);
  }

  // Fold the rotation of edge j into the running products of the levels
  // that keep it.  The entrance edge starts every level (FIRST: the
  // products are set, not multiplied into the identity).
  auto fold = [&](int j, auto first_tag) {
    constexpr bool FIRST = decltype(first_tag)::value;
    double ox, oy, oz;
    if (KIND == 0)      omega_bend(el.b, X, Px, Py, r, p, ox, oy, oz);
    else if (KIND == 4) omega_dipole(el.tp.h, el.tp.eta_h, X, Px, Py, r, p, ox, oy, oz);
    else                omega_straight(el.q.k1 * Y, el.q.k1 * X, Px, Py, r, p, ox, oy, oz);
    const double om2 = fma(ox, ox, fma(oy, oy, oz * oz));
    // Level m keeps this edge when 2^m divides j, with step w 2^m ds: the
    // rotation about Ω by 2^m times the finest angle, i.e. the finest
    // quaternion squared m times.
    const bool end_edge = j == 0 || j == N;
    if constexpr (spin32) {
      const double f = (end_edge ? 0.5 : 1.0) * ds;
      float d, sf;
      rot_deviation_f32(0.25 * f * f * om2, d, sf);
      float vx = sf * (float)(f * ox), vy = sf * (float)(f * oy), vz = sf * (float)(f * oz);
      qc_update(C0, d, vx, vy, vz);
      if (K >= 1 && (j & 1) == 0) {
        dev_square(d, vx, vy, vz);
        qc_update(C1, d, vx, vy, vz);
        if (K >= 2 && (j & 3) == 0) {
          dev_square(d, vx, vy, vz);
          qc_update(C2, d, vx, vy, vz);
          if (K >= 3 && (j & 7) == 0) {
            dev_square(d, vx, vy, vz);
            qc_update(C3, d, vx, vy, vz);
          }
        }
      }
    } else {
      // half angle θ/2 = hw |Ω|: q = (cos θ/2, sin(θ/2)/(θ/2) hw Ω)
      double c, sc;
      rot_half_series<NT, KIND == 1 || KIND == 2 || KIND == 3>((end_edge ? el.hw2_end : el.hw2_in) * om2,
                                                                  a.ymax, c, sc);
      const double g = sc * (end_edge ? el.hw_end : el.hw_in);
      Quat qb = {c, g * ox, g * oy, g * oz};
      Q0 = FIRST ? qb : qmul(qb, Q0);
      if (K >= 1 && (j & 1) == 0) {
        qb = qsquare(qb);
        Q1 = FIRST ? qb : qmul(qb, Q1);
        if (K >= 2 && (j & 3) == 0) {
          qb = qsquare(qb);
          Q2 = FIRST ? qb : qmul(qb, Q2);
          if (K >= 3 && (j & 7) == 0) {
            qb = qsquare(qb);
            Q3 = FIRST ? qb : qmul(qb, Q3);
          }
        }
      }
    }
  };

  int j0 = 0;
  if constexpr (PEEL) {
    fold(0, std::true_type{});
    j0 = 1;
  }
#pragma unroll
  for (int j = j0; j <= N; ++j) {
    if (j > 0) {
      if (KIND == 0) {
        bend_step<false>(el.b, el.b.slice, BendLane{0.0, 0.0}, X, Px, Py, Y, T, W, r, wme, Pa2,
                         invPa2);
      } else {
        series_step(all_closed, [&](auto closed, bool& beyond) {
          constexpr bool CLOSED = decltype(closed)::value;
          if constexpr (KIND == 4) teapot_slice<CLOSED>(el.tp, X, Px, Y, Py, T, p, beyond);
          else if constexpr (Y4)   quad_slice4<KIND, CLOSED>(el.q4, mc, mc0, X, Px, Y, Py, T, p, a, beyond);
          else if constexpr (MK)   mk_slice<KIND, CLOSED>(el.q, ml, X, Px, Y, Py, tk, p, beyond);
          else                     quad_step2<KIND, CLOSED>(el.q, mc, X, Px, Y, Py, T, p, a, beyond);
        }, X, Px, Y, Py, T, tk);
        if constexpr (MK) invariant(j == N ? 0.5 : 1.0);
        ps2 = p.P2() - fma(Px, Px, Py * Py);
        r = rsqrt_omega(ps2);
      }
    }
    fold(j, std::false_type{});
  }
  if (KIND == 0)
    bend_yt(el.b, el.b.whole, bend_lane(el.b, el.b.whole, p), Px_in, W_in, Px, W, Py, Y, T, invPa2);
  if constexpr (MK) T += mk_flight(ds, N, esum, fma(X, Px, Y * Py) - xp_in, tk, p);
  if constexpr (spin32) {
    Q0 = qc_to_double(C0);
    if (K >= 1) Q1 = qc_to_double(C1);
    if (K >= 2) Q2 = qc_to_double(C2);
    if (K >= 3) Q3 = qc_to_double(C3);
  }

  // Romberg tableau (§4.3 eq. romberg) with levels indexed by stride 2^m:
  // V_j[m] = (4^j V_{j-1}[m] - V_{j-1}[m+1]) / (4^j - 1), limit V_K[0].
  if (K >= 1) {
    Q0 = qextrapolate(Q0, Q1, 4.0);
    if (K >= 2) {
      Q1 = qextrapolate(Q1, Q2, 4.0);
      if (K >= 3) Q2 = qextrapolate(Q2, Q3, 4.0);
      Q0 = qextrapolate(Q0, Q1, 16.0);
      if (K >= 3) {
        Q1 = qextrapolate(Q1, Q2, 16.0);
        Q0 = qextrapolate(Q0, Q1, 64.0);
      }
    }
  }
  const double inv = rsqrt_near_one(fma(Q0.w, Q0.w, fma(Q0.x, Q0.x, fma(Q0.y, Q0.y, Q0.z * Q0.z))));
  return {Q0.w * inv, Q0.x * inv, Q0.y * inv, Q0.z * inv};
}

// ---------------------------------------------------------------------------
// Short-series bodies of sector bends and second-order quadrupoles with the slice
// counts and rows of the standard rings (lattice_table.h: the records, and the bounds
// of a lane).  The kernel is bound by VALU issue, so what counts is the instructions
// per slice edge.  With u = (Px² + Py²)/P² <= 2^-16 (bends) or 2^-14 known for the
// whole element,
//   P/Ps = 1 + u/2 + 3u²/8 + 5u³/16   and, in a bend with Pα² = P² - Py²,
//   Ps - Pα = -(v Pα)(1/2 + v/8 + v²/16), v = Px²/Pα²,
// take the place of the estimate, Newton steps and reciprocal of every edge;
// Ω is formed already scaled by half the slice length, so that the quaternion
// series gives its rotation directly; and Q is returned without its common
// factor and norm (the caller's composition is normalised as a whole).
//
// A wave in which some lane is outside the bounds runs the same body with the rest of
// the series, whose terms are multiplied by that lane's `more` (WIDE): the lanes
// inside get the same bits either way, and the others' series reach slopes of 2^-4.5,
// closed forms beyond (`rare`).  As a second body for the lanes outside it cost such
// waves twice the time: 65536 protons on the RHIC-scale ring without sextupoles, four
// times the spread, 3.0 ms a turn against 1.5 with a third of it.
// Weight of level m in the limit V_K[0] of the tableau (romberg, below the
// general body), relative to that of level 0.
template <int K>
struct RombergWeights {
  double r[K + 1];
  constexpr RombergWeights() : r{} {
    double v[K + 1][K + 1] = {};               // v[m]: V_j[m] over the levels
    for (int m = 0; m <= K; ++m) v[m][m] = 1.0;
    double c = 1.0;
    for (int j = 1; j <= K; ++j) {
      c *= 4.0;
      for (int m = 0; m + j <= K; ++m)
        for (int l = 0; l <= K; ++l) v[m][l] = (c * v[m][l] - v[m + 1][l]) / (c - 1.0);
    }
    for (int l = 0; l <= K; ++l) r[l] = v[0][l] / v[0][0];
  }
};

// Level products over the slice edges of an element with NS slices and KS + 1
// rows, from o = (ds/2) Ω: TERMS series terms, or single precision (S32).
// SPIN false: the orbit only.  WIDE: lanes outside the element's bounds (more = 1, 0
// in the others) add the rest of the launch's NT terms, or halve the angle beyond
// ymax.
template <int NT, int TERMS, int NS, int KS, bool S32, bool SPIN, bool WIDE>
struct SpinLevels {
  static_assert(KS >= 0 && KS < kMaxRows && NS % (1 << KS) == 0, "NS slices divisible by 2^KS");
  Quat q[KS + 1];
  QuatC c[KS + 1];
  double more, ymax;

  __device__ __forceinline__ SpinLevels(double more_, double ymax_) : more(more_), ymax(ymax_) {
    if constexpr (S32)
      for (int m = 0; m <= KS; ++m) c[m] = qc_ident();
  }
  __device__ __forceinline__ void fold(int j, double ox, double oy, double oz) {
    if constexpr (!SPIN) return;
    const bool end = j == 0 || j == NS;
    const double y = (end ? 0.25 : 1.0) * fma(ox, ox, fma(oy, oy, oz * oz));
    if constexpr (S32) {
      float d, sf;
      rot_deviation_f32(y, d, sf);
      if (!end) sf *= 2.0f;
      float vx = sf * (float)ox, vy = sf * (float)oy, vz = sf * (float)oz;
#pragma unroll
      for (int m = 0; m <= KS; ++m) {
        if (j % (1 << m) != 0) break;
        if (m > 0) dev_square(d, vx, vy, vz);
        qc_update(c[m], d, vx, vy, vz);
      }
    } else {
      double cs, sc;
      cos_sinc_series<TERMS>(y, cs, sc);
      if constexpr (WIDE && TERMS < NT) {
        double ct, st;
        cos_sinc_tail<NT, TERMS>(y, ct, st);
        static_assert(TERMS == 4);
        const double y2 = y * y, y4 = (more * y2) * y2;
        cs = fma(y4, ct, cs);
        sc = fma(y4, st, sc);
      }
      if constexpr (WIDE) rare(!(y <= ymax), [&] { halving_series<NT, false>(y, ymax, cs, sc); });
      if (end) sc *= 0.5;
      Quat e = {cs, sc * ox, sc * oy, sc * oz};
#pragma unroll
      for (int m = 0; m <= KS; ++m) {
        if (j % (1 << m) != 0) break;
        if (m > 0) {                            // twice the angle of a unit quaternion
          const double tw = 2.0 * e.w;
          e = {fma(tw, e.w, -1.0), tw * e.x, tw * e.y, tw * e.z};
        }
        q[m] = j == 0 ? e : qmul(e, q[m]);
      }
    }
  }
  // V_K[0] over its weight of level 0
  __device__ __forceinline__ Quat limit() {
    if constexpr (!SPIN) return Quat{};
    constexpr RombergWeights<KS> w{};
    if constexpr (S32)
      for (int m = 0; m <= KS; ++m) q[m] = qc_to_double(c[m]);
    Quat v = q[0];
#pragma unroll
    for (int m = 1; m <= KS; ++m) {
      v.w = fma(w.r[m], q[m].w, v.w);
      v.x = fma(w.r[m], q[m].x, v.x);
      v.y = fma(w.r[m], q[m].y, v.y);
      v.z = fma(w.r[m], q[m].z, v.z);
    }
    return v;
  }
};

// F = Ps - Pα and G = Pα/Ps - 1 at a bend's edge, v = Px²/Pα².  G needs its third
// term: 5v³/16 is 1e-15 at the bound, a quarter of which a passage of a few rad
// would carry into the spin.
struct BendEdge {
  double F, G;
};
template <bool WIDE>
__device__ __forceinline__ BendEdge fast_bend_edge(double Px, double invPa, const Particle& p,
                                                   double more) {
  const double t = Px * Px * invPa, v = t * invPa;
  BendEdge e = {-t * fma(v, fma(v, 0.0625, p.k18), 0.5), v * fma(v, fma(v, 0.3125, p.k38), 0.5)};
  if constexpr (WIDE) {
    const double v2 = v * v, w = more * v2;    // the terms up to v = kPsMaxU
    e.F = fma(-t * v * w, fma(v, fma(v, 21.0 / 1024.0, 7.0 / 256.0), 5.0 / 128.0), e.F);
    e.G = fma(w * v2, fma(v, 63.0 / 256.0, 35.0 / 128.0), e.G);
    rare(!(v <= kPsMaxU), [&] {
      const double r = rsqrt_nr(1.0 - v), q = rcp_nr(fma(1.0 - v, r, 1.0));   // Pα/Ps, Pα/(Pα + Ps)
      e.F = -t * q;
      e.G = v * r * q;
    });
  }
  return e;
}

// Without spin the bend is crossed in one step.
template <int NT, int NS, int KS, bool S32, bool SPIN, bool WIDE>
__device__ __forceinline__ Quat fast_bend(const HotBend& el, double& X, double& Px, double& Y,
                                          double& Py, double& T, const Particle& p, double ymax,
                                          double more) {
  SpinLevels<NT, NT, NS, KS, S32, SPIN, WIDE> lev(more, ymax);
  const double cs = SPIN ? el.cs : el.w_cs, sn = SPIN ? el.sn : el.w_sn;
  const double omc = SPIN ? el.omc : el.w_omc;
  const double w = Py * Py * p.invP2(), Pa2 = fma(-Py, Py, p.P2());
  const double dPa = p.invP * (w * fma(w, fma(w, 0.3125, p.k38), 0.5));
  double invPa = p.invP + dPa, invPa_lo = ((p.invP - invPa) + dPa) + p.invP_lo;
  if constexpr (WIDE)
    rare(!(w <= kFastBendU), [&] {
      invPa = rsqrt_nr(Pa2);
      invPa_lo = rsqrt_rest(fma(-Py, Py, p.c3), invPa);
    });
  const double Pa = Pa2 * invPa;
  BendEdge at = fast_bend_edge<WIDE>(Px, invPa, p, more);
  const double Px_in = Px, F_in = at.F;
  double wme = (el.one_m_eta2 + ((p.c3 - Py * Py) - Px * Px)) * rcp_nr((Pa + F_in) + el.eta);
  const double b = p.a2() * Py * p.invP2();                     // Ω without its path factor
  const double kf = el.hw_eta_h * invPa, ka = fma(-b, Py, p.a1());
  const double ky = kf * ka, kx = kf * b, kz = el.hw_eta_h * b;
  // ky turns the spin by Gγ times the bend, and is the same at every edge: what
  // its factors' rounding left out joins hw_h (the path factor of ky is near 1)
  const double kf_lo = fma(el.hw_eta_h, invPa_lo, fma(el.hw_eta_h, invPa, -kf));
  const double hw_h = el.hw_h - fma(kf_lo, ka, fma(kf, ka, -ky));
#pragma unroll
  for (int j = 0; j <= (SPIN ? NS : 1); ++j) {
    if (j > 0) {
      const double A = fma(-el.eta_h, X, wme), F0 = at.F;
      const double px1 = fma(Px, cs, A * sn);
      at = fast_bend_edge<WIDE>(px1, invPa, p, more);
      const double dW = at.F - F0;
      X = fma(X, cs, fma(wme, omc, fma(Px, sn, dW)) * el.inv_eta_h);
      wme += dW;
      Px = px1;
    }
    const double path = fma(el.h, X, 1.0);
    const double g = fma(path, at.G, path);                    // path Pα/Ps
    lev.fold(j, (g * kx) * Px, fma(-g, ky, hw_h), path * kz);
  }
  // the slices' angle differences telescope; |sin| < 0.008 in the bounds.  Ps = Pα +
  // F: 1/Pα enters once, since its rounding is the same in every bend and T follows it
  const double sd = ((Px_in - Px) + fma(Px_in, at.F * invPa, -Px * (F_in * invPa))) * invPa;
  const double s2 = sd * sd;
  double D = fma(sd * s2, fma(s2, fma(s2, AC<3>::v, AC<2>::v), AC<1>::v), sd);
  if constexpr (WIDE) rare(!(fabs(sd) <= 0.0078125), [&] { D = asin_small(sd); });
  Y = fma(Py, fma(D, el.inv_eta_h, el.s_eta), Y);
  T += fma(-(p.ib() * el.inv_eta_h), D, fma(-p.Pt, el.s_eta, el.tconst));
  return lev.limit();
}

// Whether a lane is inside the bounds of the element's short series (HotBend,
// HotQuad).  The conditions are combined without branches.
__device__ __forceinline__ bool fast_lane(const Record& r, double X, double Px, double Y,
                                          double Py, const Particle& p) {
  bool in = fabs(p.c3) <= kFastC3;
  if (r.op < OP_MKX) {
    const HotBend& f = r.b;
    in &= fma(f.turn_x, fabs(X), fma(f.turn_c, fabs(p.c3), fabs(Px))) <= f.mom;
    in &= fabs(Py) <= kFastMom;
    in &= fabs(X) <= f.x_max;
  } else {
    const HotQuad& f = r.q;
    const double R = fabs(X) + fabs(Y), Q = fabs(Px) + fabs(Py);
    in &= fma(f.mom_x, R, f.mom_p * Q) <= 2.0 * kFastMom;
    in &= fma(f.reach, Q, R) <= f.x_max;
  }
  return in;
}

// (ds/2) Ω at an edge of a quadrupole: rho = P/Ps, ka = -(ds/2) k1 a1/P,
// kg = (ds/2) k1 a2/P².
__device__ __forceinline__ void fast_quad_omega(double ka, double kg, double invP, double rho,
                                                double X, double Px, double Y, double Py,
                                                double& ox, double& oy, double& oz) {
  oz = kg * fma(Px, Y, Py * X);
  const double k = oz * invP;
  ox = rho * fma(ka, Y, k * Px);
  oy = rho * fma(ka, X, k * Py);
}

// Four terms cover the half angle up to kFastQuadAngle: y^4/8! < 2^-56.
constexpr int kFastQuadTerms = 4;

// P/Ps - 1 from u = (Px² + Py²)/P².
template <bool WIDE>
__device__ __forceinline__ double fast_quad_e(double u, double Px, double Py, const Particle& p,
                                              double more) {
  double e = u * fma(u, fma(u, 0.3125, p.k38), 0.5);
  if constexpr (WIDE) {
    const double u2 = u * u;                   // the terms up to u = kPsMaxU
    e = fma((more * u2) * u2, fma(u, 63.0 / 256.0, 35.0 / 128.0), e);
    rare(!(u <= kPsMaxU), [&] {
      const double ps2 = p.P2() - fma(Px, Px, Py * Py), r = rsqrt_nr(ps2);
      e = u * (p.P() * r) * rcp_nr(fma(ps2 * r, p.invP, 1.0));
    });
  }
  return e;
}

// Matrix-kick quadrupole (KIND 1 focusing in x, 3 in y).
template <int NT, int KIND, int NS, int KS, bool S32, bool SPIN, bool WIDE>
__device__ __forceinline__ Quat fast_mk(const HotQuad& el, double& X, double& Px, double& Y,
                                        double& Py, double& T, const Particle& p, MKCache* mkc,
                                        double ymax, double more) {
  SpinLevels<NT, kFastQuadTerms, NS, KS, S32, SPIN, WIDE> lev(more, ymax);
  const MKLin m = mk_cached(el.q, p, mkc);
  const double ka = -el.hw_k1 * p.a1() * p.invP, kg = el.hw_k1 * p.a2() * p.invP2();
  const double kP = fabs(el.q.k1) * p.P(), xp_in = fma(X, Px, Y * Py);
  const double dsp = el.q.ds * p.invP;
  double esum = 0.0, tk = 0.0;
#pragma unroll
  for (int j = 0; j <= NS; ++j) {
    if (j > 0) {
      if (KIND == 1) mk_move(m, X, Px, Y, Py);
      else           mk_move(m, Y, Py, X, Px);
      const double u = fma(Px, Px, Py * Py) * p.invP2(), u2 = u * u;
      const double e = fast_quad_e<WIDE>(u, Px, Py, p, more);
      const double d = dsp * e;                                // ds (1/Ps - 1/P)
      X = fma(Px, d, X);
      Y = fma(Py, d, Y);
      const double tk0 = tk;
      tk = fma(u2, fma(u, 0.21875, p.k14), tk);                // g - u (u/2 + g)/4
      if constexpr (WIDE) {
        tk = fma((more * u2) * u2, fma(u, 91.0 / 512.0, 25.0 / 128.0), tk);
        rare(!(u <= kPsMaxU), [&] {
          // g = u² (2 + ρ)/(2ρ (1 + ρ)²), ρ = Ps/P = 1/(1 + e)
          const double rho1 = 1.0 + rcp_nr(1.0 + e);           // 1 + Ps/P
          const double g = u2 * (1.0 + rho1) * (1.0 + e) * 0.5 * rcp_nr(rho1 * rho1);
          tk = tk0 + fma(-0.25 * u, e, g);
        });
      }
      if (KIND == 1) mk_move(m, X, Px, Y, Py);
      else           mk_move(m, Y, Py, X, Px);
    }
    const double pp = fma(Px, Px, Py * Py);
    const double inv = KIND == 1 ? mk_invariant(kP, pp, X, Y) : mk_invariant(kP, pp, Y, X);
    esum = (j == 0 || j == NS) ? fma(0.5, inv, esum) : esum + inv;
    const double rho = 1.0 + fast_quad_e<WIDE>(pp * p.invP2(), Px, Py, p, more);
    double ox, oy, oz;
    fast_quad_omega(ka, kg, p.invP, rho, X, Px, Y, Py, ox, oy, oz);
    lev.fold(j, ox, oy, oz);
  }
  T += mk_flight(el.q.ds, NS, esum, fma(X, Px, Y * Py) - xp_in, tk, p);
  return lev.limit();
}

// Drift-kick-drift quadrupole: the two half drifts that meet at an interior
// edge have the same momenta, which Ω at that edge uses too.
template <int NT, int NS, int KS, bool S32, bool SPIN, bool WIDE>
__device__ __forceinline__ Quat fast_dkd(const HotQuad& el, double& X, double& Px, double& Y,
                                         double& Py, double& T, const Particle& p, double ymax,
                                         double more) {
  SpinLevels<NT, kFastQuadTerms, NS, KS, S32, SPIN, WIDE> lev(more, ymax);
  const double ka = -el.hw_k1 * p.a1() * p.invP, kg = el.hw_k1 * p.a2() * p.invP2();
  double esum = 0.0, e = 0.0, c = 0.0;          // e = P/Ps - 1, c = (ds/2)/Ps
#pragma unroll
  for (int j = 0; j <= NS; ++j) {
    if (j > 0) {
      X = fma(c, Px, X);
      Y = fma(c, Py, Y);
      Px = fma(-el.q.k1ds, X, Px);
      Py = fma(el.q.k1ds, Y, Py);
    }
    const double u = fma(Px, Px, Py * Py) * p.invP2();
    const double e0 = e;
    e = fast_quad_e<WIDE>(u, Px, Py, p, more);
    if (j > 0) esum += e0;
    c = el.q.hds * fma(p.invP, e, p.invP);
    if (j > 0) {
      X = fma(c, Px, X);
      Y = fma(c, Py, Y);
      esum += e;
    }
    double ox, oy, oz;
    fast_quad_omega(ka, kg, p.invP, 1.0 + e, X, Px, Y, Py, ox, oy, oz);
    lev.fold(j, ox, oy, oz);
  }
  T -= fma(el.q.hds * p.invbeta(), esum, (NS * el.q.ds) * p.dib);
  return lev.limit();
}

// Orbit only through a thick element (surrogate tracking, no spin): the
// sector bend is an exact flow and is crossed in one step; quadrupoles keep
// their slices, and matrix-kick ones take their constants from the lane's
// cache when one is passed.
template <int KIND, bool Y4 = false>
__device__ __forceinline__ void thick_orbit(const DevElem& el, double& X, double& Px, double& Y,
                                            double& Py, double& T, const Particle& p,
                                            const TrackArgs& a, MKCache* mkc = nullptr) {
  if (KIND == 0) {
    const double Pa2 = p.P2() - Py * Py;
    const double ps2 = fma(-Px, Px, Pa2);
    double r = rsqrt_nr(ps2);
    double W = ps2 * r;
    double wme = (el.b.one_m_eta2 + ((p.c3 - Py * Py) - Px * Px)) * rcp_nr(W + el.b.eta);
    bend_step(el.b, el.b.whole, bend_lane(el.b, el.b.whole, p), X, Px, Py, Y, T, W, r, wme, Pa2,
              rcp_nr(Pa2));
    return;
  }
  if constexpr (Y4) {
    MKConst m1, m0;
    if (KIND == 1 || KIND == 3) { m1 = mk_const(el.q4.s1, p); m0 = mk_const(el.q4.s0, p); }
    for (int j = 0; j < el.nsl; ++j)
      series_step(false, [&](auto closed, bool& beyond) {
        quad_slice4<KIND, decltype(closed)::value>(el.q4, m1, m0, X, Px, Y, Py, T, p, a, beyond);
      }, X, Px, Y, Py, T);
    return;
  }
  if constexpr (KIND == 1 || KIND == 3) {
    const MKLin ml = mk_cached(el.q, p, mkc);
    const double kP = fabs(el.q.k1) * p.P(), xp_in = fma(X, Px, Y * Py);
    double esum = 0.0, tk = 0.0;
    for (int j = 0; j <= el.nsl; ++j) {
      if (j > 0)
        series_step(false, [&](auto closed, bool& beyond) {
          mk_slice<KIND, decltype(closed)::value>(el.q, ml, X, Px, Y, Py, tk, p, beyond);
        }, X, Px, Y, Py, tk);
      const double pp = fma(Px, Px, Py * Py);
      esum = fma(j == 0 || j == el.nsl ? 0.5 : 1.0,
                 KIND == 1 ? mk_invariant(kP, pp, X, Y) : mk_invariant(kP, pp, Y, X), esum);
    }
    T += mk_flight(el.q.ds, el.nsl, esum, fma(X, Px, Y * Py) - xp_in, tk, p);
    return;
  }
  for (int j = 0; j < el.nsl; ++j)
    series_step(KIND == 4 && el.tp.closed != 0.0, [&](auto closed, bool& beyond) {
      constexpr bool CLOSED = decltype(closed)::value;
      if constexpr (KIND == 4) teapot_slice<CLOSED>(el.tp, X, Px, Y, Py, T, p, beyond);
      else quad_step2<KIND, CLOSED>(el.q, MKConst{}, X, Px, Y, Py, T, p, a, beyond);
    }, X, Px, Y, Py, T);
}

// Piece-wise constant spin through a thick element (§4.1 eq. pwcSpin): one
// rotation by ds·Ω per slice, later slices on the left, Ω taken between the
// two half kicks of a drift-kick slice (PLACE == P_KICK; KIND 2 or 4) or at
// the middle of the slice (P_MIDPOINT: the element carries 2N orbit half
// slices and the rotation lies between the two of a slice).
template <int NT, int KIND, int PLACE, bool Y4 = false>
__device__ __forceinline__ Quat pwc_element(const DevElem& el, double& X, double& Px, double& Y,
                                            double& Py, double& T, const Particle& p,
                                            const TrackArgs& a) {
  const double ds_orb = KIND == 0 ? el.b.ds : (KIND == 4 ? el.tp.ds : el.q.ds);
  const double w = PLACE == P_MIDPOINT ? 2.0 * ds_orb : ds_orb;   // spin step
  Quat Q = qident();
  MKConst mc, mc0;
  if constexpr (Y4) {
    if (KIND == 1 || KIND == 3) { mc = mk_const(el.q4.s1, p); mc0 = mk_const(el.q4.s0, p); }
  } else {
    if (KIND == 1 || KIND == 3) mc = mk_const(el.q, p);
  }
  double Pa2 = 0.0, invPa2 = 0.0, W = 0.0, r = 0.0, wme = 0.0;
  BendLane bl{0.0, 0.0};
  if (KIND == 0) {
    bl = bend_lane(el.b, el.b.slice, p);
    Pa2 = p.P2() - Py * Py;
    invPa2 = rcp_nr(Pa2);
    const double ps2 = fma(-Px, Px, Pa2);
    r = rsqrt_nr(ps2);
    W = ps2 * r;
    wme = (el.b.one_m_eta2 + ((p.c3 - Py * Py) - Px * Px)) * rcp_nr(W + el.b.eta);
  }
  // drift-kick half slices: the two drifts that meet between kicks have the
  // same momenta, which Ω there uses too
  constexpr bool DKD = KIND == 2 && PLACE == P_MIDPOINT && !Y4;
  PsInv ps{0.0, 0.0};
  double esum = 0.0;
  if constexpr (DKD) {
    const double pp = fma(Px, Px, Py * Py);
    series_step(false, [&](auto closed, bool& beyond) {
      ps = ps_part<decltype(closed)::value>(pp, p, beyond);
    });
  }
  // half of a slice (P_MIDPOINT), or of its drift and kick, entered or left (P_KICK)
  auto half = [&](auto closed, bool& beyond, bool leave) {
    constexpr bool CLOSED = decltype(closed)::value;
    if constexpr (DKD) {
      double c = el.q.hds * ps.r;
      X = fma(c, Px, X);
      Y = fma(c, Py, Y);
      esum += ps.e;
      Px = fma(-el.q.k1ds, X, Px);
      Py = fma(el.q.k1ds, Y, Py);
      ps = ps_part<CLOSED>(fma(Px, Px, Py * Py), p, beyond);
      c = el.q.hds * ps.r;
      X = fma(c, Px, X);
      Y = fma(c, Py, Y);
      esum += ps.e;
    } else if constexpr (PLACE == P_KICK && KIND == 4) {
      if (!leave) teapot_drift<CLOSED>(el.tp, X, Px, Y, Py, T, p, beyond);
      teapot_kick(el.tp, 0.5 * el.tp.ds, X, Px);
      if (leave) teapot_drift<CLOSED>(el.tp, X, Px, Y, Py, T, p, beyond);
    } else if constexpr (PLACE == P_KICK) {
      if (!leave) drift_part<CLOSED>(el.q.hds, X, Px, Y, Py, T, p, a.inv_beta0, beyond);
      Px = fma(-0.5 * el.q.k1ds, X, Px);
      Py = fma(0.5 * el.q.k1ds, Y, Py);
      if (leave) drift_part<CLOSED>(el.q.hds, X, Px, Y, Py, T, p, a.inv_beta0, beyond);
    } else if constexpr (KIND == 0) {
      bend_step<true, CLOSED>(el.b, el.b.slice, bl, X, Px, Py, Y, T, W, r, wme, Pa2, invPa2, &beyond);
    } else if constexpr (KIND == 4) {
      teapot_slice<CLOSED>(el.tp, X, Px, Y, Py, T, p, beyond);
    } else if constexpr (Y4) {
      quad_slice4<KIND, CLOSED>(el.q4, mc, mc0, X, Px, Y, Py, T, p, a, beyond);
    } else {
      quad_step2<KIND, CLOSED>(el.q, mc, X, Px, Y, Py, T, p, a, beyond);
    }
  };
  const int slices = PLACE == P_MIDPOINT ? el.nsl / 2 : el.nsl;
  for (int j = 0; j < slices; ++j) {
    double ox, oy, oz;
    series_step(KIND == 4 && el.tp.closed != 0.0, [&](auto closed, bool& beyond) {
      constexpr bool CLOSED = decltype(closed)::value;
      half(closed, beyond, false);
      double ri = r;
      if constexpr (DKD) ri = ps.r;
      else if constexpr (KIND != 0)
        ri = ps_part<CLOSED>(fma(Px, Px, Py * Py), p, beyond).r;
      if (KIND == 0)      omega_bend(el.b, X, Px, Py, ri, p, ox, oy, oz);
      else if (KIND == 4) omega_dipole(el.tp.h, el.tp.eta_h, X, Px, Py, ri, p, ox, oy, oz);
      else                omega_straight(el.q.k1 * Y, el.q.k1 * X, Px, Py, ri, p, ox, oy, oz);
      half(closed, beyond, true);
    }, X, Px, Y, Py, T, W, r, wme, ps.r, ps.e, esum);
    double c, sfac;
    rot_half_angle<NT, KIND == 1 || KIND == 2 || KIND == 3>(
        0.25 * w * w * fma(ox, ox, fma(oy, oy, oz * oz)), a.ymax, c, sfac);
    const double g = sfac * w;
    Q = qmul(Quat{c, g * ox, g * oy, g * oz}, Q);
  }
  if constexpr (DKD)
    T -= el.q.hds * fma(p.invbeta(), esum, 2.0 * el.nsl * p.dib);
  const double inv = rsqrt_near_one(fma(Q.w, Q.w, fma(Q.x, Q.x, fma(Q.y, Q.y, Q.z * Q.z))));
  return {Q.w * inv, Q.x * inv, Q.y * inv, Q.z * inv};
}

// Solenoid (§3.7, §4.4): entrance fringe kick, body slices with the spin at
// the slice edges (Romberg) or at the slice middles (PLACE == P_MIDPOINT: 2N
// orbit half slices), exit fringe kick; later rotations on the left.
template <int NT, int PLACE>
__device__ __forceinline__ Quat solenoid_element(const DevElem& el, double& X, double& Px,
                                                 double& Y, double& Py, double& T,
                                                 const Particle& p, const TrackArgs& a) {
  const SolenoidParams& sp = el.sol;
  auto rot = [&](double wx, double wy, double wz) {
    double c, sfac;
    rot_half_angle<NT, true>(0.25 * fma(wx, wx, fma(wy, wy, wz * wz)), a.ymax, c, sfac);
    return Quat{c, sfac * wx, sfac * wy, sfac * wz};
  };
  double wx, wy, wz;
  solenoid_fringe(sp, 1.0, X, Px, Y, Py, p, wx, wy, wz);
  const Quat qin = rot(wx, wy, wz);
  const SolState st = sol_state<NT>(sp, X, Px, Y, Py, p, a.ymax, a.inv_beta0);
  Quat Q;
  if (PLACE == P_MIDPOINT) {
    Q = qident();
    const double w = 2.0 * sp.ds;
    for (int j = 1; j <= el.nsl; ++j) {
      solenoid_slice(sp, st, X, Px, Y, Py, T);
      if (j & 1) {
        double ox, oy, oz;
        omega_solenoid(sp, st, X, Px, Y, Py, p, ox, oy, oz);
        Q = qmul(rot(w * ox, w * oy, w * oz), Q);
      }
    }
  } else {
    // Romberg levels over the slice edges, as for the other thick elements
    const int N = el.nsl, K = el.K;
    const double ds = sp.ds;
    Quat Q0 = qident(), Q1 = qident(), Q2 = qident(), Q3 = qident();
    for (int j = 0; j <= N; ++j) {
      if (j > 0) solenoid_slice(sp, st, X, Px, Y, Py, T);
      double ox, oy, oz;
      omega_solenoid(sp, st, X, Px, Y, Py, p, ox, oy, oz);
      const double f = ((j == 0 || j == N) ? 0.5 : 1.0) * ds;
      Quat qb = rot(f * ox, f * oy, f * oz);
      Q0 = qmul(qb, Q0);
      if (K >= 1 && (j & 1) == 0) {
        qb = qsquare(qb);
        Q1 = qmul(qb, Q1);
        if (K >= 2 && (j & 3) == 0) {
          qb = qsquare(qb);
          Q2 = qmul(qb, Q2);
          if (K >= 3 && (j & 7) == 0) {
            qb = qsquare(qb);
            Q3 = qmul(qb, Q3);
          }
        }
      }
    }
    if (K >= 1) {
      Q0 = qextrapolate(Q0, Q1, 4.0);
      if (K >= 2) {
        Q1 = qextrapolate(Q1, Q2, 4.0);
        if (K >= 3) Q2 = qextrapolate(Q2, Q3, 4.0);
        Q0 = qextrapolate(Q0, Q1, 16.0);
        if (K >= 3) {
          Q1 = qextrapolate(Q1, Q2, 16.0);
          Q0 = qextrapolate(Q0, Q1, 64.0);
        }
      }
    }
    Q = Q0;
  }
  const double inv = rsqrt_near_one(fma(Q.w, Q.w, fma(Q.x, Q.x, fma(Q.y, Q.y, Q.z * Q.z))));
  Q = {Q.w * inv, Q.x * inv, Q.y * inv, Q.z * inv};
  solenoid_fringe(sp, -1.0, X, Px, Y, Py, p, wx, wy, wz);
  return qmul(rot(wx, wy, wz), qmul(Q, qin));
}

// Rectangular bend (§3.2, §4.5): frame rotation by φ^entr into the magnet
// (the spin components turn with the frame about ŷ), entrance fringe and its
// spin kick, body slices with Romberg over the edges or midpoint rotations,
// X referred to the design orbit's exit point (eq. Xoffset), exit fringe and
// kick, frame rotation by -φ^exit out; T referred to the design arc (eq.
// Toffset).
template <int NT, int PLACE>
__device__ __forceinline__ Quat rbend_element(const DevElem& el, double& X, double& Px, double& Y,
                                              double& Py, double& T, const Particle& p,
                                              const TrackArgs& a) {
  const RbendParams& rb = el.rb;
  auto rot = [&](double wx, double wy, double wz) {
    double c, sfac;
    rot_half_angle<NT>(0.25 * fma(wx, wx, fma(wy, wy, wz * wz)), a.ymax, c, sfac);
    return Quat{c, sfac * wx, sfac * wy, sfac * wz};
  };
  // fringe kick ±fb Y [G(γ - 1) Px x̂ - (1 + G) ẑ]
  auto fringe_spin = [&](double sign) {
    const double f = sign * rb.fb * Y;
    const double wx = f * p.a2() * Px, wz = -f * (1.0 + a.G);
    double c, sfac;
    rot_half_angle<NT, true>(0.25 * fma(wx, wx, wz * wz), a.ymax, c, sfac);
    return Quat{c, sfac * wx, 0.0, sfac * wz};
  };
  rbend_rotate(rb.in, X, Px, Y, Py, T, p);
  rbend_fringe(rb, 1.0, X, Px, Y, Py, T, p);
  const Quat qin = fringe_spin(1.0);
  Quat Q;
  auto omega_at = [&](double& ox, double& oy, double& oz) {
    const double r = rsqrt_nr(p.P2() - fma(Px, Px, Py * Py));
    omega_dipole(0.0, rb.fb, X, Px, Py, r, p, ox, oy, oz);
  };
  if (PLACE == P_MIDPOINT) {
    Q = qident();
    const double w = 2.0 * rb.ds;
    for (int j = 1; j <= el.nsl; ++j) {
      rbend_body(rb, rb.ds, X, Px, Y, Py, T, p);
      if (j & 1) {
        double ox, oy, oz;
        omega_at(ox, oy, oz);
        Q = qmul(rot(w * ox, w * oy, w * oz), Q);
      }
    }
  } else {
    const int N = el.nsl, K = el.K;
    Quat Q0 = qident(), Q1 = qident(), Q2 = qident(), Q3 = qident();
    for (int j = 0; j <= N; ++j) {
      if (j > 0) rbend_body(rb, rb.ds, X, Px, Y, Py, T, p);
      double ox, oy, oz;
      omega_at(ox, oy, oz);
      const double f = ((j == 0 || j == N) ? 0.5 : 1.0) * rb.ds;
      Quat qb = rot(f * ox, f * oy, f * oz);
      Q0 = qmul(qb, Q0);
      if (K >= 1 && (j & 1) == 0) {
        qb = qsquare(qb);
        Q1 = qmul(qb, Q1);
        if (K >= 2 && (j & 3) == 0) {
          qb = qsquare(qb);
          Q2 = qmul(qb, Q2);
          if (K >= 3 && (j & 7) == 0) {
            qb = qsquare(qb);
            Q3 = qmul(qb, Q3);
          }
        }
      }
    }
    if (K >= 1) {
      Q0 = qextrapolate(Q0, Q1, 4.0);
      if (K >= 2) {
        Q1 = qextrapolate(Q1, Q2, 4.0);
        if (K >= 3) Q2 = qextrapolate(Q2, Q3, 4.0);
        Q0 = qextrapolate(Q0, Q1, 16.0);
        if (K >= 3) {
          Q1 = qextrapolate(Q1, Q2, 16.0);
          Q0 = qextrapolate(Q0, Q1, 64.0);
        }
      }
    }
    Q = Q0;
  }
  const double inv = rsqrt_near_one(fma(Q.w, Q.w, fma(Q.x, Q.x, fma(Q.y, Q.y, Q.z * Q.z))));
  Q = {Q.w * inv, Q.x * inv, Q.y * inv, Q.z * inv};
  X -= rb.xoff;
  const Quat qout = fringe_spin(-1.0);
  rbend_fringe(rb, -1.0, X, Px, Y, Py, T, p);
  rbend_rotate(rb.out, X, Px, Y, Py, T, p);
  T += rb.larc_ib0;
  const Quat qfi = {rb.in.qw, 0.0, rb.in.qy, 0.0}, qfo = {rb.out.qw, 0.0, rb.out.qy, 0.0};
  return qmul(qfo, qmul(qout, qmul(Q, qmul(qin, qfi))));
}

// Spin kick across the thin fringe of a normal 2m-pole face crossed about
// normally (§4.5 eq. skfringe): a rotation about ẑ by
// -sign (1 + G) (b_m/(Bρ)0) Im[(X + iY)^m]/m, sign +1 at the entrance.
// Sector bends (KIND 0, 4) are m = 1 with b1/(Bρ)0 = ηh; quadrupoles m = 2
// with b2/(Bρ)0 = k1.
template <int NT, int KIND>
__device__ __forceinline__ Quat fringe_kick(const DevElem& el, double X, double Y, double sign,
                                            const TrackArgs& a) {
  const double im = (KIND == 0) ? el.b.eta_h * Y : (KIND == 4) ? el.tp.eta_h * Y : el.q.k1 * X * Y;
  const double w = -sign * (1.0 + a.G) * im;
  double c, sfac;
  rot_half_angle<NT, true>(0.25 * w * w, a.ymax, c, sfac);
  return Quat{c, 0.0, 0.0, sfac * w};
}

// Spin and orbit of a thick element with the extended methods: TEAPOT bends,
// the piece-wise constant placements and the fringe spin kicks.
template <int NT, int KIND, bool Y4>
__device__ __forceinline__ Quat thick_body_ext(const DevElem& el, double& X, double& Px, double& Y,
                                            double& Py, double& T, const Particle& p,
                                            const TrackArgs& a) {
  if (el.place == P_KICK) {   // one kick per slice: not with the composed slices
    if constexpr (!Y4 && (KIND == 2 || KIND == 4))
      return pwc_element<NT, KIND, P_KICK>(el, X, Px, Y, Py, T, p, a);
    return qident();   // rejected on the host
  }
  if (el.place == P_MIDPOINT)
    return pwc_element<NT, KIND, P_MIDPOINT, Y4>(el, X, Px, Y, Py, T, p, a);
  return thick_element<NT, KIND, false, Y4, false>(el, X, Px, Y, Py, T, p, a);
}

// The body between the fringe spin kicks of its faces (elements flagged
// F_FRINGE): q_exit · Q_body · q_entrance.
template <int NT, int KIND, bool Y4>
__device__ __forceinline__ Quat thick_ext_y(const DevElem& el, double& X, double& Px, double& Y,
                                         double& Py, double& T, const Particle& p,
                                         const TrackArgs& a) {
  if (!(el.flags & F_FRINGE)) return thick_body_ext<NT, KIND, Y4>(el, X, Px, Y, Py, T, p, a);
  const Quat qin = fringe_kick<NT, KIND>(el, X, Y, 1.0, a);
  const Quat Q = thick_body_ext<NT, KIND, Y4>(el, X, Px, Y, Py, T, p, a);
  return qmul(fringe_kick<NT, KIND>(el, X, Y, -1.0, a), qmul(Q, qin));
}

template <int NT, int KIND>
__device__ __forceinline__ Quat thick_ext(const DevElem& el, double& X, double& Px, double& Y,
                                       double& Py, double& T, const Particle& p,
                                       const TrackArgs& a) {
  if constexpr (KIND == 1 || KIND == 2 || KIND == 3) {
    if (el.orbit == M_DKD4 || el.orbit == M_MK4)
      return thick_ext_y<NT, KIND, true>(el, X, Px, Y, Py, T, p, a);
  }
  return thick_ext_y<NT, KIND, false>(el, X, Px, Y, Py, T, p, a);
}

template <int NT>
__device__ __forceinline__ Quat thin_element(const ThinParams& e, double X, double& Px, double Y,
                                             double& Py, const Particle& p, const TrackArgs& a) {
  const double hk1 = 0.5 * e.k1l, hk2 = 0.5 * e.k2l;
  Px -= fma(hk1, X, 0.5 * hk2 * (X * X - Y * Y));
  Py += fma(hk1, Y, hk2 * X * Y);
  double ps2 = p.P2() - fma(Px, Px, Py * Py);
  double r = rsqrt_omega(ps2);
  double bx = fma(e.k2l * X, Y, e.k1l * Y);
  double by = fma(e.k1l, X, 0.5 * e.k2l * (X * X - Y * Y));
  double ox, oy, oz;
  omega_straight(bx, by, Px, Py, r, p, ox, oy, oz);
  const double y = 0.25 * fma(ox, ox, fma(oy, oy, oz * oz));
  Px -= fma(hk1, X, 0.5 * hk2 * (X * X - Y * Y));
  Py += fma(hk1, Y, hk2 * X * Y);
  double c, sfac;
  rot_half_angle<NT, true>(y, a.ymax, c, sfac);
  return {c, sfac * ox, sfac * oy, sfac * oz};
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// The short-series body of a record (op from OP_BEND83 on).
template <int NT, bool S32, bool SPIN, bool WIDE>
__device__ __forceinline__ Quat fast_thick(const Record& r, double& X, double& Px, double& Y,
                                           double& Py, double& T, const Particle& p, MKCache* mkc,
                                           double ymax, double more) {
  if (r.op == OP_MKX) return fast_mk<NT, 1, 4, 2, S32, SPIN, WIDE>(r.q, X, Px, Y, Py, T, p, mkc, ymax, more);
  if (r.op == OP_MKY) return fast_mk<NT, 3, 4, 2, S32, SPIN, WIDE>(r.q, X, Px, Y, Py, T, p, mkc, ymax, more);
  if (r.op == OP_BEND83) return fast_bend<NT, 8, 3, S32, SPIN, WIDE>(r.b, X, Px, Y, Py, T, p, ymax, more);
  if (r.op == OP_DKD82) return fast_dkd<NT, 8, 2, S32, SPIN, WIDE>(r.q, X, Px, Y, Py, T, p, ymax, more);
  return fast_bend<NT, 8, 2, S32, SPIN, WIDE>(r.b, X, Px, Y, Py, T, p, ymax, more);
}

// The general body of a sector bend or a second-order quadrupole with the spin
// at the slice edges.
template <int NT, bool S32, bool SPIN>
__device__ __forceinline__ Quat general_thick(const DevElem& e, double& X, double& Px, double& Y,
                                              double& Py, double& T, const Particle& p,
                                              const TrackArgs& a, MKCache* mkc) {
  if constexpr (SPIN) {
    if (e.kind == K_SBEND)    return thick_element<NT, 0, S32>(e, X, Px, Y, Py, T, p, a);
    if (e.orbit != M_MK)      return thick_element<NT, 2, S32>(e, X, Px, Y, Py, T, p, a);
    if (e.q.k1 >= 0.0)        return thick_element<NT, 1, S32>(e, X, Px, Y, Py, T, p, a, mkc);
    return thick_element<NT, 3, S32>(e, X, Px, Y, Py, T, p, a, mkc);
  } else {
    if (e.kind == K_SBEND)    thick_orbit<0>(e, X, Px, Y, Py, T, p, a);
    else if (e.orbit != M_MK) thick_orbit<2>(e, X, Px, Y, Py, T, p, a);
    else if (e.q.k1 >= 0.0)   thick_orbit<1>(e, X, Px, Y, Py, T, p, a, mkc);
    else                      thick_orbit<3>(e, X, Px, Y, Py, T, p, a, mkc);
    return Quat{};
  }
}

// Elements of the extended kernels (OP_EXT).
template <int NT>
__device__ __forceinline__ Quat ext_element(const DevElem& e, double& X, double& Px, double& Y,
                                            double& Py, double& T, const Particle& p,
                                            const TrackArgs& a) {
  if (e.kind == K_RBEND) {
    if (e.place == P_MIDPOINT) return rbend_element<NT, P_MIDPOINT>(e, X, Px, Y, Py, T, p, a);
    return rbend_element<NT, P_EDGES>(e, X, Px, Y, Py, T, p, a);
  }
  if (e.kind == K_SOLENOID) {
    if (e.place == P_MIDPOINT) return solenoid_element<NT, P_MIDPOINT>(e, X, Px, Y, Py, T, p, a);
    return solenoid_element<NT, P_EDGES>(e, X, Px, Y, Py, T, p, a);
  }
  if (e.kind == K_SBEND) {
    if (e.orbit == M_TEAPOT) return thick_ext<NT, 4>(e, X, Px, Y, Py, T, p, a);
    return thick_ext<NT, 0>(e, X, Px, Y, Py, T, p, a);
  }
  if (e.orbit == M_DKD || e.orbit == M_DKD4) return thick_ext<NT, 2>(e, X, Px, Y, Py, T, p, a);
  if (e.q.k1 >= 0.0) return thick_ext<NT, 1>(e, X, Px, Y, Py, T, p, a);
  return thick_ext<NT, 3>(e, X, Px, Y, Py, T, p, a);
}

template <int NT>
__device__ __forceinline__ void ext_orbit(const DevElem& e, double& X, double& Px, double& Y,
                                          double& Py, double& T, const Particle& p,
                                          const TrackArgs& a) {
  if (e.kind == K_RBEND) {
    rbend_rotate(e.rb.in, X, Px, Y, Py, T, p);
    rbend_fringe(e.rb, 1.0, X, Px, Y, Py, T, p);
    rbend_body(e.rb, e.rb.L, X, Px, Y, Py, T, p);
    X -= e.rb.xoff;
    rbend_fringe(e.rb, -1.0, X, Px, Y, Py, T, p);
    rbend_rotate(e.rb.out, X, Px, Y, Py, T, p);
    T += e.rb.larc_ib0;
  } else if (e.kind == K_SOLENOID) {
    const SolState st = sol_state<NT>(e.sol, X, Px, Y, Py, p, a.ymax, a.inv_beta0);
    for (int jj = 0; jj < e.nsl; ++jj) solenoid_slice(e.sol, st, X, Px, Y, Py, T);
  } else if (e.kind == K_SBEND) {
    if (e.orbit == M_TEAPOT) thick_orbit<4>(e, X, Px, Y, Py, T, p, a);
    else                     thick_orbit<0>(e, X, Px, Y, Py, T, p, a);
  } else if (e.orbit == M_DKD4) {
    thick_orbit<2, true>(e, X, Px, Y, Py, T, p, a);
  } else if (e.orbit == M_MK4) {
    if (e.q.k1 >= 0.0) thick_orbit<1, true>(e, X, Px, Y, Py, T, p, a);
    else               thick_orbit<3, true>(e, X, Px, Y, Py, T, p, a);
  } else if (e.orbit == M_DKD) {
    thick_orbit<2>(e, X, Px, Y, Py, T, p, a);
  } else if (e.q.k1 >= 0.0) {
    thick_orbit<1>(e, X, Px, Y, Py, T, p, a);
  } else {
    thick_orbit<3>(e, X, Px, Y, Py, T, p, a);
  }
}

// One record's element: the state moves through it, and its quaternion is
// returned (ORBIT: not formed).  A caller that drops one of the two leaves its
// arithmetic to dead-code elimination and gets the same bits in the other.
template <int NT, bool MIXED, bool EXT, bool ORBIT>
__device__ __forceinline__ Quat element_pass(const Record& r, const ConstElem* tab, double& X,
                                             double& Px, double& Y, double& Py, double& T,
                                             const Particle& p, const TrackArgs& a, MKCache* mkc) {
  Quat q;
  if (r.op >= OP_THICK) {
    // the mixed kernel carries both precisions; an element runs one
    const bool s32 = MIXED && (r.flags & F_SPIN32);
    // (extended kernels: the general bodies only.  With the short-series ones in them
    // the slice loops of their own elements ran up to 12 % slower, drift-kick bends
    // with midpoint spin, 8 slices, 100003 particles, 1894 us for four turns against
    // 1697; a ring with one solenoid gains 16 % from them, 262144 particles.)
    if (!EXT && r.op > OP_THICK) {
      const bool in = fast_lane(r, X, Px, Y, Py, p);
      if (__all(in)) {
        if (s32) q = fast_thick<NT, MIXED, !ORBIT, false>(r, X, Px, Y, Py, T, p, mkc, a.ymax, 0.0);
        else     q = fast_thick<NT, false, !ORBIT, false>(r, X, Px, Y, Py, T, p, mkc, a.ymax, 0.0);
      } else {
        const double more = in ? 0.0 : 1.0;
        if (s32) q = fast_thick<NT, MIXED, !ORBIT, true>(r, X, Px, Y, Py, T, p, mkc, a.ymax, more);
        else     q = fast_thick<NT, false, !ORBIT, true>(r, X, Px, Y, Py, T, p, mkc, a.ymax, more);
      }
    } else {
      const DevElem e = load_elem(tab + r.elem);
      if (s32) q = general_thick<NT, MIXED, !ORBIT>(e, X, Px, Y, Py, T, p, a, mkc);
      else     q = general_thick<NT, false, !ORBIT>(e, X, Px, Y, Py, T, p, a, mkc);
    }
  } else if (EXT && r.op == OP_EXT) {
    const DevElem e = load_elem(tab + r.elem);
    if (ORBIT) ext_orbit<NT>(e, X, Px, Y, Py, T, p, a);
    else       q = ext_element<NT>(e, X, Px, Y, Py, T, p, a);
  } else if (r.op == OP_THIN) {
    if (ORBIT) {
      const double hk1 = 0.5 * r.t.k1l, hk2 = 0.5 * r.t.k2l;
      for (int h = 0; h < 2; ++h) {
        Px -= fma(hk1, X, 0.5 * hk2 * (X * X - Y * Y));
        Py += fma(hk1, Y, hk2 * X * Y);
      }
    } else {
      q = thin_element<NT>(r.t, X, Px, Y, Py, p, a);
    }
  } else {
    q = {r.s.qw, r.s.qx, r.s.qy, r.s.qz};
  }
  return q;
}

// A block's LDS: cold per-lane data, the spin (touched once per turn) and the
// orbit at the current element's entrance (read back only on a loss).
struct BlockShared {
  double cold[8][kBlock];
  double mk_slot[kMKWords][kBlock];
  double red[kBlock / 64][4];   // (last: the lanes' addresses start at 0; 4 to 8 % of an extended turn)
};

// EXT: the kernel also knows the drift-kick sector bend, the piece-wise
// constant spin placements, solenoids and rectangular bends (kept out of the
// other instantiations so that their register allocation is not shaped by code
// they never run).
// ORBIT: the network turns of the particles on the network, the first
// a.feat_n lanes of the lane order: the orbit only, with the network's inputs
// written at the start of each turn.
template <int NT, bool MIXED, bool EXT, bool ORBIT>
__device__ __forceinline__ void track_body(const TrackArgs& a, int block, BlockShared& sh) {
  auto& red = sh.red;
  auto& cold = sh.cold;
  auto& mk_slot = sh.mk_slot;
  const int tid = threadIdx.x;
  const int64_t g = a.lane0 + (int64_t)block * kBlock + tid;
  const bool valid = g < a.lane0 + a.n_lanes;
  const int64_t j = (valid && a.perm) ? (int64_t)a.perm[g] : g;
  int32_t status = valid ? a.alive[j] : 0;
  bool live = status == 1;
  const int64_t n = a.n;

  double X = 0, Px = 0, Y = 0, Py = 0, T = 0, Pt = 0;
  cold[0][tid] = 0.0; cold[1][tid] = 0.0; cold[2][tid] = 0.0;
  if (valid) {
    X = a.z[j]; Px = a.z[n + j]; Y = a.z[2 * n + j]; Py = a.z[3 * n + j];
    T = a.z[4 * n + j]; Pt = a.z[5 * n + j];
    cold[0][tid] = a.spin[j]; cold[1][tid] = a.spin[n + j]; cold[2][tid] = a.spin[2 * n + j];
  }
  // Without reports the kernel has no barrier, so a wave with no live lane
  // (a replay of a few particles) may leave at once.
  if (a.report_every == 0 && !__any(live)) {
    if (ORBIT && a.turns_done && valid) a.turns_done[g] = 0;
    return;
  }
  const Particle p = make_particle(Pt, a);
  MKCache mkc{&mk_slot[0][tid], kBlock, __builtin_nan(""), __builtin_nan("")};
  Quat qturn = qident();
  // The lattice is read-only for the whole launch: reading it through the
  // constant address space lets the uniform loads go through the scalar cache.
  const ConstElem* tab = (const ConstElem*)(a.tab);
  const ConstRecord* rec = (const ConstRecord*)(a.rec);
  const ConstSeq* seq = (const ConstSeq*)(a.seq);

  int turns_done = 0;
  for (int t = 1; t <= a.turns; ++t) {
    const bool was_live = live;
    if (was_live) qturn = qident();
    if (ORBIT && a.feat && live) {
      // the network's inputs at the start of this turn
      float* f = a.feat + ((int64_t)(t - 1) * a.feat_n + g) * a.feat_n_in;
      f[0] = (float)((X - a.feat_center[0]) * a.feat_inv_scale[0]);
      f[1] = (float)((Px - a.feat_center[1]) * a.feat_inv_scale[1]);
      f[2] = (float)((Y - a.feat_center[2]) * a.feat_inv_scale[2]);
      f[3] = (float)((Py - a.feat_center[3]) * a.feat_inv_scale[3]);
      f[4] = (float)((T - a.feat_center[4]) * a.feat_inv_scale[4]);
      f[5] = (float)((Pt - a.feat_center[5]) * a.feat_inv_scale[5]);
      if (a.feat_n_in == 7) f[6] = (float)a.feat_extra;
    }
    // A record is loaded while the one before it finishes (its loss check, the
    // composition and the drift behind it), and its index one record earlier:
    // loaded where they were used, the four dependent scalar loads of a record
    // took a lone wave 0.59 of 3.0 million cycles a turn on the RHIC-scale ring.
    Record r = load_record(rec + seq[0]);
    uint32_t next = seq[min(1, a.n_records)];
    int ie = 0;                  // lattice index of the record's first element
    for (int ir = 0; ir < a.n_records; ++ir) {
      const int op = r.op, flags = r.flags, count = r.count;
      const double tail = r.tail;
      Quat q;
      if (live && op != OP_NONE) {
        cold[3][tid] = X; cold[4][tid] = Px; cold[5][tid] = Y; cold[6][tid] = Py;
        cold[7][tid] = T;
        q = element_pass<NT, MIXED, EXT, ORBIT>(r, tab, X, Px, Y, Py, T, p, a, &mkc);
      }
      r = load_record(rec + next);
      next = seq[min(ir + 2, a.n_records)];
      if (live) {
        if (op != OP_NONE) {
          bool ok = fabs(X) <= a.aperture;
          ok &= fabs(Y) <= a.aperture;
          ok &= isfinite(Px);
          ok &= isfinite(Py);
          ok &= isfinite(T);
          if (!ok) {
            X = cold[3][tid]; Px = cold[4][tid]; Y = cold[5][tid]; Py = cold[6][tid];
            T = cold[7][tid];
            live = false;
            status = -(1 + ie);
          } else if (!ORBIT) {
            qturn = qmul(q, qturn);
          }
        }
        if ((flags & F_TAIL) && live) {
          cold[3][tid] = X; cold[5][tid] = Y; cold[7][tid] = T;
          drift(tail, X, Px, Y, Py, T, p, a.inv_beta0);
          bool ok = fabs(X) <= a.aperture;
          ok &= fabs(Y) <= a.aperture;
          ok &= isfinite(T);
          if (!ok) {
            X = cold[3][tid]; Y = cold[5][tid]; T = cold[7][tid];
            live = false;
            status = -(ie + count);
          }
        }
      }
      ie += count;
      // the short-series bodies leave their common factor (0.69 or more) in
      if (!ORBIT && (ir & 31) == 31 && was_live) qturn = qnormalized(qturn);
    }
    if (was_live && live) ++turns_done;
    // A particle lost during this turn still receives the rotation of the
    // elements it completed before the loss.
    double sx = cold[0][tid], sy = cold[1][tid], sz = cold[2][tid];
    if (!ORBIT && was_live) {
      qturn = qnormalized(qturn);
      qrotate(qturn, sx, sy, sz);
      cold[0][tid] = sx; cold[1][tid] = sy; cold[2][tid] = sz;
    }
    if (a.report_every > 0 && t % a.report_every == 0) {
      double v0 = live ? sx : 0.0, v1 = live ? sy : 0.0, v2 = live ? sz : 0.0;
      double v3 = live ? 1.0 : 0.0;
      v0 = wave_sum(v0); v1 = wave_sum(v1); v2 = wave_sum(v2); v3 = wave_sum(v3);
      const int lane = tid & 63, wv = tid >> 6;
      if (lane == 0) { red[wv][0] = v0; red[wv][1] = v1; red[wv][2] = v2; red[wv][3] = v3; }
      __syncthreads();
      if (tid < 4) {
        double s = 0.0;
        for (int k = 0; k < kBlock / 64; ++k) s += red[k][tid];
        const int rep = t / a.report_every - 1;
        a.partials[((int64_t)rep * a.n_blocks + block) * 4 + tid] = s;
      }
      __syncthreads();
    }
  }

  if (ORBIT && a.turns_done && valid) a.turns_done[g] = turns_done;
  if (valid && a.alive[j] == 1) {
    a.z[j] = X; a.z[n + j] = Px; a.z[2 * n + j] = Y; a.z[3 * n + j] = Py; a.z[4 * n + j] = T;
    if (!ORBIT) {
      a.spin[j] = cold[0][tid]; a.spin[n + j] = cold[1][tid]; a.spin[2 * n + j] = cold[2][tid];
    }
    a.alive[j] = status;
    if (a.qout) {
      a.qout[j] = qturn.w; a.qout[n + j] = qturn.x; a.qout[2 * n + j] = qturn.y;
      a.qout[3 * n + j] = qturn.z;
    }
  }
}

template <int NT, bool MIXED, bool EXT>
__global__ void __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu((MIXED || EXT) ? ST_WAVES_PER_EU_WIDE : ST_WAVES_PER_EU)))
track_kernel(const TrackArgs a) {
  __shared__ BlockShared sh;
  track_body<NT, MIXED, EXT, false>(a, blockIdx.x, sh);
}

// Without the spin arithmetic the orbit push fits 123 registers, so four waves
// share a SIMD (the LDS of their workgroups fits a CU); with the extended elements
// it is two.
template <int NT, bool EXT>
__global__ void __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(EXT ? 2 : ST_WAVES_PER_EU_ORBIT)))
orbit_kernel(const TrackArgs a) {
  __shared__ BlockShared sh;
  track_body<NT, false, EXT, true>(a, blockIdx.x, sh);
}

}  // namespace

template <bool MIXED, bool EXT>
static hipError_t launch_nt(const TrackArgs& a, int nt, hipStream_t stream) {
  const dim3 grid((unsigned)a.n_blocks), block(kBlock);
  switch (nt) {
    case 5:  hipLaunchKernelGGL((track_kernel<5, MIXED, EXT>), grid, block, 0, stream, a); break;
    case 6:  hipLaunchKernelGGL((track_kernel<6, MIXED, EXT>), grid, block, 0, stream, a); break;
    case 8:  hipLaunchKernelGGL((track_kernel<8, MIXED, EXT>), grid, block, 0, stream, a); break;
    case 9:  hipLaunchKernelGGL((track_kernel<9, MIXED, EXT>), grid, block, 0, stream, a); break;
    case 12: hipLaunchKernelGGL((track_kernel<12, MIXED, EXT>), grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL((track_kernel<16, MIXED, EXT>), grid, block, 0, stream, a); break;
  }
  return hipGetLastError();
}

}  // namespace st
