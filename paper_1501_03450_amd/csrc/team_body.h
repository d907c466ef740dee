// Teams of four waves per 64 particles, on the element loop of track_body.h.
#pragma once

#include "track_body.h"

namespace st {
namespace {

// Few particles (kTeamLanes).  One wave per 64 particles leaves most of the chip
// idle, and a turn is one wave's chain (RHIC-scale ring: 1.25 ms, of which the
// vector instructions issue 62 %).  Only the orbit has to go through the
// elements in order; an element's quaternion needs the state at its entrance
// alone.  So a team of four waves, one per SIMD of a compute unit, shares 64
// particles: wave 0 pushes the orbits and leaves the entrance states of a batch
// of elements in LDS; waves 1 to 3 take elements of the batch before, recompute
// the slices and form the quaternions; wave 1 composes those of the batch before
// that in lattice order, and turns the spins.  Every step ends in a barrier.
// The arithmetic is element_pass's and the order of composition the lattice's,
// so the results are those of track_kernel bit for bit.  333 particles: 1249 -> 818
// us a turn; 1024 on the small ring: 117 -> 71 us.  What bounds it now is wave 0:
// a dependent double-precision FMA takes 7.6 cycles here where independent ones
// issue every 4.6; seven waves to form quaternions instead of three gain nothing.
// Extended elements gain as much: 32 bends and 32 quadrupoles in 8 slices, teams of
// 1657 particles against one round of blocks, us a turn: drift-kick with the spin at
// the kicks 152 / 227, fourth-order drift-kick quadrupoles 140 / 278, matrix-kick
// ones 180 / 319.
constexpr int kTeam = 64;              // particles of a team
constexpr int kTeamBatch = 8;          // elements of a batch
constexpr int kTeamWaves = 4;
constexpr int kComposeCost = 3;

struct TeamMeta {
  uint64_t live, ok;       // lanes alive at the element's entrance and after its loss check
  int32_t rec, ir;         // the record and its place in the sequence
  int32_t who;             // the wave that forms its quaternion
};

struct TeamShared {
  double entry[2][kTeamBatch][4][kTeam];      // X, Px, Y, Py
  double quat[2][kTeamBatch][4][kTeam];
  double mk_slot[kTeamWaves][kMKWords][kTeam];
  double cold_t[kTeam];
  TeamMeta meta[2][kTeamBatch], qmeta[2][kTeamBatch];
  int32_t filled[2], last[2];
  uint64_t end_live[2];
};

template <int NT, bool EXT>
__device__ __forceinline__ void team_body(const TrackArgs& a, int block, TeamShared& sh) {
  auto& entry = sh.entry;
  auto& quat = sh.quat;
  auto& mk_slot = sh.mk_slot;
  auto& cold_t = sh.cold_t;
  auto& meta = sh.meta;
  auto& qmeta = sh.qmeta;
  auto& filled = sh.filled;
  auto& last = sh.last;
  auto& end_live = sh.end_live;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t g = a.lane0 + (int64_t)block * kTeam + lane, n = a.n;
  const bool valid = g < a.lane0 + a.n_lanes;
  const int64_t j = (valid && a.perm) ? (int64_t)a.perm[g] : g;
  const int32_t status0 = valid ? a.alive[j] : 0;
  const bool live0 = status0 == 1;
  // every wave sees the same statuses here, so all leave or none
  if (a.report_every == 0 && !__any(live0)) return;
  const ConstElem* tab = (const ConstElem*)(a.tab);
  const ConstRecord* rec = (const ConstRecord*)(a.rec);
  const ConstSeq* seq = (const ConstSeq*)(a.seq);
  const Particle p = make_particle(valid ? a.z[5 * n + j] : 0.0, a);
  MKCache mkc{&mk_slot[wave][0][lane], kTeam, __builtin_nan(""), __builtin_nan("")};
  int buf = 0;               // the buffer that the next batch goes to

  if (wave == 0) {
    double X = 0, Px = 0, Y = 0, Py = 0, T = 0;
    if (valid) {
      X = a.z[j]; Px = a.z[n + j]; Y = a.z[2 * n + j]; Py = a.z[3 * n + j]; T = a.z[4 * n + j];
    }
    bool live = live0;
    int32_t status = status0;
    for (int t = 1; t <= a.turns; ++t) {
      Record r = load_record(rec + seq[0]);
      int32_t cur = seq[0], next = seq[min(1, a.n_records)];
      int ie = 0, ir = 0;
      bool done = false;
      while (!done) {
        int k = 0;
        int load[kTeamWaves] = {};
        load[1] = kComposeCost;                 // wave 1 composes as well
        for (; ir < a.n_records && k < kTeamBatch; ++ir) {
          const int op = r.op, flags = r.flags, count = r.count;
          const double tail = r.tail;
          const uint64_t at_entry = __ballot(live);
          double (*en)[kTeam] = entry[buf][k];
          if (op != OP_NONE) {
            en[0][lane] = X; en[1][lane] = Px; en[2][lane] = Y; en[3][lane] = Py;
            cold_t[lane] = T;
            if (live) (void)element_pass<NT, false, EXT, false>(r, tab, X, Px, Y, Py, T, p, a, &mkc);
          }
          const int32_t now = cur;
          r = load_record(rec + next);
          cur = next;
          next = seq[min(ir + 2, a.n_records)];
          if (op != OP_NONE) {
            bool ok = fabs(X) <= a.aperture;
            ok &= fabs(Y) <= a.aperture;
            ok &= isfinite(Px);
            ok &= isfinite(Py);
            ok &= isfinite(T);
            if (live && !ok) {
              X = en[0][lane]; Px = en[1][lane]; Y = en[2][lane]; Py = en[3][lane];
              T = cold_t[lane];
              live = false;
              status = -(1 + ie);
            }
            const uint64_t after = __ballot(live);
            const int cost = EXT && op == OP_EXT ? 10 : op < OP_THICK ? 1 : op == OP_THICK ? 10 : op < OP_MKX ? 7 : 5;
            int who = 1, least = load[1];       // the wave with the least to do
#pragma unroll
            for (int w = 2; w < kTeamWaves; ++w) {
              who = load[w] < least ? w : who;
              least = min(least, load[w]);
            }
#pragma unroll
            for (int w = 1; w < kTeamWaves; ++w) load[w] += w == who ? cost : 0;
            if (lane == 0) meta[buf][k] = TeamMeta{at_entry, after, now, ir, who};
            ++k;
          }
          if ((flags & F_TAIL) && live) {
            const double X0 = X, Y0 = Y, T0 = T;
            drift(tail, X, Px, Y, Py, T, p, a.inv_beta0);
            bool ok = fabs(X) <= a.aperture;
            ok &= fabs(Y) <= a.aperture;
            ok &= isfinite(T);
            if (!ok) {
              X = X0; Y = Y0; T = T0;
              live = false;
              status = -(ie + count);
            }
          }
          ie += count;
        }
        done = ir >= a.n_records;
        const uint64_t now_live = __ballot(live);
        if (lane == 0) {
          filled[buf] = k;
          last[buf] = done;
          end_live[buf] = now_live;
        }
        __syncthreads();       // the batch is there; the one before it is consumed
        buf ^= 1;
      }
      __syncthreads();         // the last batch is consumed
    }
    if (live0) {
      a.z[j] = X; a.z[n + j] = Px; a.z[2 * n + j] = Y; a.z[3 * n + j] = Py; a.z[4 * n + j] = T;
      a.alive[j] = status;
    }
    return;
  }

  double sx = 0, sy = 0, sz = 0;
  Quat qturn = qident();
  bool was_live = live0;
  if (wave == 1 && valid) { sx = a.spin[j]; sy = a.spin[n + j]; sz = a.spin[2 * n + j]; }
  int composed = 0;            // records behind the composed product (normalised every 32)
  auto normalise_to = [&](int end) {
    for (; (composed | 31) < end; composed = (composed | 31) + 1)
      if (was_live) qturn = qnormalized(qturn);
  };
  auto compose = [&](int b, int k1) {
    for (int k = 0; k < k1; ++k) {
      const int ir = __builtin_amdgcn_readfirstlane(qmeta[b][k].ir);
      const bool ok = (qmeta[b][k].ok >> lane) & 1;
      normalise_to(ir);
      const Quat q = {quat[b][k][0][lane], quat[b][k][1][lane], quat[b][k][2][lane],
                      quat[b][k][3][lane]};
      if (ok) qturn = qmul(q, qturn);
    }
  };
  for (int t = 1; t <= a.turns; ++t) {
    if (wave == 1 && was_live) qturn = qident();
    composed = 0;
    int before = 0;            // elements of the batch before this one
    bool done = false;
    __syncthreads();           // the turn's first batch is there
    while (!done) {
      const int b = buf;
      const int k1 = __builtin_amdgcn_readfirstlane(filled[b]);
      done = __builtin_amdgcn_readfirstlane(last[b]) != 0;
      if (wave == 1) compose(b ^ 1, before);
      for (int k = 0; k < k1; ++k) {
        const TeamMeta m = meta[b][k];
        if (__builtin_amdgcn_readfirstlane(m.who) != wave) continue;
        const Record r = load_record(rec + __builtin_amdgcn_readfirstlane(m.rec));
        Quat q = qident();
        if ((m.live >> lane) & 1) {
          double X = entry[b][k][0][lane], Px = entry[b][k][1][lane];
          double Y = entry[b][k][2][lane], Py = entry[b][k][3][lane], T = 0.0;
          q = element_pass<NT, false, EXT, false>(r, tab, X, Px, Y, Py, T, p, a, &mkc);
        }
        quat[b][k][0][lane] = q.w; quat[b][k][1][lane] = q.x;
        quat[b][k][2][lane] = q.y; quat[b][k][3][lane] = q.z;
        if (lane == 0) qmeta[b][k] = m;
      }
      before = k1;
      buf ^= 1;
      __syncthreads();         // the batch is consumed; the next one, if any, is there
    }
    if (wave == 1) {
      compose(buf ^ 1, before);
      normalise_to(a.n_records);
      if (was_live) {
        qturn = qnormalized(qturn);
        qrotate(qturn, sx, sy, sz);
      }
      const bool live = (end_live[buf ^ 1] >> lane) & 1;
      if (a.report_every > 0 && t % a.report_every == 0) {
        double v[4] = {live ? sx : 0.0, live ? sy : 0.0, live ? sz : 0.0, live ? 1.0 : 0.0};
        double mine = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          v[c] = wave_sum(v[c]);
          if (lane == c) mine = v[c];
        }
        const int rep = t / a.report_every - 1;
        if (lane < 4) a.partials[((int64_t)rep * a.n_blocks + block) * 4 + lane] = mine;
      }
      was_live = live;
    }
  }
  if (wave == 1 && live0) {
    a.spin[j] = sx; a.spin[n + j] = sy; a.spin[2 * n + j] = sz;
    if (a.qout) {
      a.qout[j] = qturn.w; a.qout[n + j] = qturn.x; a.qout[2 * n + j] = qturn.y;
      a.qout[3 * n + j] = qturn.z;
    }
  }
}

template <int NT, bool EXT>
__global__ void __launch_bounds__(kTeam * kTeamWaves) __attribute__((amdgpu_waves_per_eu(2)))
team_kernel(const TrackArgs a) {
  __shared__ TeamShared sh;
  team_body<NT, EXT>(a, blockIdx.x, sh);
}

}  // namespace

template <bool EXT>
static hipError_t launch_team(const TrackArgs& a, int nt, hipStream_t stream) {
  const dim3 grid((unsigned)a.n_blocks), block(kTeam * kTeamWaves);
  switch (nt) {
    case 5:  hipLaunchKernelGGL((team_kernel<5, EXT>), grid, block, 0, stream, a); break;
    case 6:  hipLaunchKernelGGL((team_kernel<6, EXT>), grid, block, 0, stream, a); break;
    case 8:  hipLaunchKernelGGL((team_kernel<8, EXT>), grid, block, 0, stream, a); break;
    case 9:  hipLaunchKernelGGL((team_kernel<9, EXT>), grid, block, 0, stream, a); break;
    case 12: hipLaunchKernelGGL((team_kernel<12, EXT>), grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL((team_kernel<16, EXT>), grid, block, 0, stream, a); break;
  }
  return hipGetLastError();
}

}  // namespace st
