// Device-side lattice representation shared by the host setup code and the
// tracking kernels.
//
// A ring of ~1.7k elements repeats a handful of distinct magnets, so the
// lattice is stored as small tables with every per-element constant precomputed
// on the host (trigonometry of the bend angle per slice, reciprocals, snake
// quaternions), plus a 32-bit index sequence.  The kernels walk the sequence
// with wave-uniform loads, so the tables are read through the scalar cache and
// every branch on the element kind is uniform.  A record is one element with
// the drift that follows it, if one does (a ring alternates magnets and drifts,
// so this halves the records).  It holds what the standard bodies use of the
// element, in few enough words that the scalar registers take the next record
// while the current one finishes; the general bodies read the whole element
// (DevElem) where they run.
#pragma once

#include <stdint.h>

namespace st {

enum : int32_t { K_MARKER = 0, K_DRIFT = 1, K_SBEND = 2, K_QUAD = 3, K_THIN = 4, K_SNAKE = 5,
                 K_SOLENOID = 6, K_RBEND = 7 };
enum : int32_t { M_EXACT = 0, M_DKD = 1, M_MK = 2, M_TEAPOT = 3, M_DKD4 = 4, M_MK4 = 5 };
// spin placement in thick elements: Romberg over the slice edges, or one
// piece-wise constant rotation per slice between the half kicks or at the
// slice's middle
enum : int32_t { P_EDGES = 0, P_KICK = 1, P_MIDPOINT = 2 };

constexpr int kMaxRows = 4;   // Romberg tableau rows supported by the kernels

// (Px² + Py²)/P² up to which P/Ps is a series: series_g, and ps_part
constexpr double kSeriesMaxU = 1.0 / 4096.0, kPsMaxU = 1.0 / 512.0;

// Per-kind parameters, precomputed on the host.
struct BendStep {          // constants of one exact step of length s
  double cs, sn, omc;      // cos(h s), sin(h s), 1 - cos(h s)
  double s_eta;            // s / η
  double tconst;           // (1 - 1/η) s / β0
};
struct BendParams {        // sector bend (§3.1)
  double ds;               // slice length L/N
  double h, eta, eta_h, inv_eta_h;
  double one_m_eta2;       // 1 - η²
  BendStep slice;          // s = ds
  BendStep whole;          // s = L (orbit-only passes)
};
struct QuadParams {        // quadrupole (§3.3, §3.4)
  double ds, hds;          // slice length and half of it
  double k1, k1ds;         // gradient, DKD kick k1·ds
  double kabs_hds2;        // |k1| (ds/2)²: (κ ds/2)² times P
};
struct Quad4Params {       // fourth-order quadrupole slice (M_DKD4, M_MK4)
  QuadParams q;            // the whole slice (Ω weights, k1)
  QuadParams s1, s0;       // the composed steps of lengths x1 ds and x0 ds
};
struct TeapotParams {       // drift-kick sector bend (§3.6)
  double ds;                // orbit slice length (kick length)
  double h, eta_h;          // curvature and dipole field ηh
  double half;              // drift half ds/2
  double closed;            // 1: Px leaves ps_part's series inside the slices
  double c, sn, tn, sec;    // cos, sin, tan, 1/cos of h ds/2
  double tn_h, omc_h;       // tan(h ds/2)/h and (1/cos(h ds/2) - 1)/h
  double d0;                // ds/2 - tan(h ds/2)/h
};
struct SolenoidParams {     // solenoid (§3.7, §4.4)
  double ds;                // orbit slice length
  double ks;                // b0/(Bρ)0
  double eta, inv_eta;      // ks/2 and its inverse
  double eta_q;             // ks/4: half the vector potential at a fringe
};
struct RbendFace {          // frame rotation by φ at a rectangular-bend face
  double c, tn, sec;        // cos φ, tan φ, 1/cos φ
  double qw, qy;            // the spin's frame rotation (cos φ/2, sin φ/2 ŷ)
};
struct RbendParams {        // rectangular bend (§3.2, §4.5)
  double ds;                // orbit slice length along the magnet
  double L;                 // straight length (one-step orbit)
  double fb, rhob;          // b1/(Bρ)0 and its inverse
  double xoff;              // the design orbit's exit X in the magnet (eq. Xoffset)
  double larc_ib0;          // design arc length / β0 (eq. Toffset)
  RbendFace in, out;        // rotations by φ^entr and by -φ^exit
};
struct ThinParams { double k1l, k2l; };             // thin multipole (§3.5)
struct SnakeParams { double qw, qx, qy, qz; };      // fixed rotation quaternion

constexpr int kElemWords = sizeof(BendParams) / sizeof(double);   // largest member
static_assert(sizeof(TeapotParams) <= sizeof(BendParams), "element union size");
static_assert(sizeof(SolenoidParams) <= sizeof(BendParams), "element union size");
static_assert(sizeof(RbendParams) <= sizeof(BendParams), "element union size");
static_assert(sizeof(Quad4Params) <= sizeof(BendParams), "element union size");

// element flags: single-precision spin arithmetic; thin-fringe spin kicks at
// both faces (sector bends and quadrupoles, extended kernels only); a drift of
// length `tail` follows the element
enum : int32_t { F_SPIN32 = 1, F_FRINGE = 2, F_TAIL = 4 };

// What a record runs, chosen on the host.  From OP_THICK on: elements whose
// general bodies every kernel has; from OP_BEND83 on: those for which the plain and
// mixed kernels have a short-series body, whose slice loop is unrolled (sector bends
// with 8 slices and 4 or 3 rows, MK quadrupoles with 4 slices and 3 rows, focusing in
// x or in y, DKD ones with 8 slices and 3 rows: the counts of the standard rings; the
// series do not depend on them, but each pair is another body in the kernel).
enum : int32_t { OP_NONE = 0, OP_THIN = 1, OP_SNAKE = 2, OP_EXT = 3, OP_THICK = 4, OP_BEND83 = 5,
                 OP_BEND82 = 6, OP_MKX = 7, OP_MKY = 8, OP_DKD82 = 9 };

// Short-series bodies of sector bends and second-order quadrupoles: a lane is inside
// their bounds when its particle is within kFastC3 of the reference
// momentum, its transverse momenta (scaled by p0) stay below a bound through
// the element, and its offsets below one that keeps the slice rotations inside
// the quaternion series.  Both are decided at the entrance from these bounds
// on the motion inside:
// bends       |Px| + turn_c |P² - 1| + turn_x |X| <= mom (so that |Px| stays
//             below kFastMom), |Py| <= kFastMom, |X| <= x_max
//             (each of (Px/P)², (Py/P)² <= 2^-16)
// quadrupoles mom_p Q + mom_x R <= 2 kFastMom, R + reach Q <= x_max, with
//             R = |X| + |Y| and Q = |Px| + |Py|: (Px² + Py²)/P² <= 2^-14 (a
//             quadrupole's kick of 2.5 mrad at 3 cm takes 1.3 % of a Gaussian
//             bunch's passages beyond kFastMom, which would send half of the
//             waves through the wide form; 3e-6 beyond twice that)
constexpr double kFastC3 = 0.125;       // |P² - 1|
constexpr double kFastMom = 0.0036;     // below 2^-8 sqrt(1 - kFastC3)
constexpr double kFastQuadAngle = 0.029; // half the slice rotation of a quadrupole edge
constexpr double kFastBendU = 0x1p-16;   // range of the series of 1/Pα in Py²/P²

struct DevElem {
  int32_t kind, orbit, nsl, K;   // K = R_e - 1: Romberg levels minus one
  int32_t flags, place;          // place: P_EDGES, P_KICK or P_MIDPOINT (nsl = 2N orbit
                                 // half slices for P_MIDPOINT)
  // Romberg edge rotations of sliced elements: half the step w ds of an end
  // edge (w = 1/2) and of an interior edge (w = 1), and their squares
  double hw_end, hw_in, hw2_end, hw2_in;
  union {
    BendParams b;
    TeapotParams tp;
    SolenoidParams sol;
    RbendParams rb;
    QuadParams q;
    Quad4Params q4;
    ThinParams t;
    SnakeParams s;
    double v[kElemWords];
  };
};

struct HotBend {           // short-series sector bend (OP_BEND83, OP_BEND82)
  double cs, sn, omc;      // one slice
  double h, eta_h, inv_eta_h, eta, one_m_eta2;
  double s_eta, tconst;    // the whole bend
  double x_max, mom, turn_c, turn_x;
  double hw_eta_h, hw_h;   // (ds/2) η h and (ds/2) h
  double w_cs, w_sn, w_omc;  // the whole bend (orbit-only passes)
};
struct HotQuad {           // short-series quadrupole (OP_MKX, OP_MKY, OP_DKD82)
  QuadParams q;
  double hw_k1;            // (ds/2) k1
  double x_max, mom_p, mom_x, reach;
};
constexpr int kHotWords = sizeof(HotBend) / sizeof(double);
static_assert(sizeof(HotQuad) <= sizeof(HotBend), "record size");

struct Record {
  int32_t op, flags;
  int32_t count;           // lattice elements of the record (1 or 2)
  int32_t elem;            // index of the element in the table of elements
  double tail;             // length of the drift after the element (F_TAIL); a drift by itself is
                           // OP_NONE with a tail
  union {
    HotBend b;
    HotQuad q;
    ThinParams t;
    SnakeParams s;
    double v[kHotWords];
  };
};

struct TrackArgs {
  double* z;          // 6 × n SoA
  double* spin;       // 3 × n SoA
  int32_t* alive;     // n
  double* qout;       // 4 × n SoA or null
  int64_t n;
  const Record* rec;
  const DevElem* tab;
  const uint32_t* seq;   // n_records indices and one more, 0 (read ahead, not used)
  int32_t n_records;
  int32_t turns;
  int32_t report_every;
  int32_t n_blocks;   // set by the launch
  double* partials;   // [n_reports][n_blocks][4]
  double beta0, inv_beta0, gamma0, inv_gamma0_sq, G, aperture;
  double ymax;        // largest (θ/2)² the quaternion polynomial covers
  int64_t lane0, n_lanes;  // lanes of the launch in the lane order
  // optional lane order: lane g works on particle perm[g] (a permutation of
  // 0..n-1), so that particles taking the same path share waves
  const int32_t* perm;
  // orbit-only launches: the particles on the network are lanes g < feat_n
  // (the lane order puts them first); such a lane writes its network inputs at
  // the start of every turn, feat[(turn * feat_n + g) * feat_n_in + i] =
  // (z_i - center_i) * inv_scale_i (i < 6) and extra (i = 6), and the number of
  // turns it completes alive, turns_done[g]
  float* feat;
  int32_t* turns_done;
  int64_t feat_n;
  int32_t feat_n_in;
  double feat_center[6], feat_inv_scale[6], feat_extra;
};

}  // namespace st
