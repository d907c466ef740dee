// Launchers of the tracking kernels (host side).
#pragma once

#include <hip/hip_runtime.h>

#include "lattice_table.h"

namespace st {

int track_block_size();
int team_size();

// How a launch runs.  nt: number of series terms of the double-precision
// quaternion half-angle series (5, 6, 8, 9, 12, 16); mixed: the kernel with
// single-precision spin arithmetic in the elements flagged for it; ext: the
// lattice uses drift-kick (TEAPOT) bends, piece-wise constant spin placements,
// solenoids or rectangular bends (run in double precision); team: four waves
// per 64 particles (not in mixed precision), the same results bit for bit.
struct TrackPlan {
  int nt;
  bool mixed, ext, team;
};
// Lanes up to which a team per 64 particles is the faster one: its extra work
// (the slices are computed twice) fills SIMDs that would idle.  Two teams fit a
// compute unit, so this is one round of them; past it a second round starts, and
// the blocks take the same time up to 65536 lanes.  Teams against blocks (those of
// 32832 lanes), us a turn: RHIC-scale ring 810 / 1252 at 16384 lanes and 1030 / 1252
// at 32768; the small ring 104 / 147 at 32768.
constexpr int64_t kTeamLanes = 32768;

// Tracks a.n_lanes lanes from a.lane0 on, in blocks of 256 lanes or teams of 64
// (the polarization partials have that many rows per report).
hipError_t launch_track(TrackArgs a, const TrackPlan& plan, hipStream_t stream);

// Surrogate tracking: the orbit only of the orbit.feat_n particles on the network
// (the first lanes of the lane order), and the turns of the fallback ones.  Where
// those are few enough for teams and the orbits for kBesideLanes, one launch runs
// both beside each other: each is a chain that leaves SIMDs idle.
hipError_t launch_surrogate_turns(TrackArgs orbit, TrackArgs fallback, const TrackPlan& plan,
                                  hipStream_t stream);
// Orbit lanes of one round in that launch, whose registers (the teams') leave two
// waves per SIMD; the orbit kernel of its own has four.
constexpr int64_t kBesideLanes = 131072;

hipError_t launch_surrogate_spin(double* spin, const int32_t* alive, const int32_t* fallback,
                                 const float* qnn, int64_t n, hipStream_t s);
// Network rotations of a multi-turn surrogate launch for the n_net particles
// on the network, lanes g < n_net of the lane order perm (qnn [turn][n_net][4]
// and turns_done [n_net] from the launch).
hipError_t launch_surrogate_spin_turns(double* spin, const int32_t* perm,
                                       const int32_t* turns_done, const float* qnn, int64_t n_net,
                                       int64_t n, hipStream_t s);
// Audit of the network quaternions against the tracked ones: failures get
// fallback[j] = turn and failed[j] = 1; every other particle failed[j] = 0.
hipError_t launch_audit(const int32_t* alive, int32_t* fallback, int32_t* failed, const float* qnn,
                        const double* q64, int64_t n, double threshold, int32_t turn,
                        hipStream_t s);
// Rollback to the checkpoint, and status after the replay, of the particles
// with failed[j] != 0.
hipError_t launch_replay_prepare(const int32_t* failed, double* z, double* spin,
                                 const double* ck_z, const double* ck_spin, const int32_t* ck_alive,
                                 int32_t* ralive, int64_t n, hipStream_t s);
hipError_t launch_replay_finish(const int32_t* failed, const int32_t* ralive, int32_t* alive,
                                int64_t n, hipStream_t s);
// Lane order for surrogate tracking: a stable partition of 0..n-1 (see
// partition_key; flag is the audit's failed[] array in mode 1); counts and
// offsets hold 3 ints per 256 particles.
hipError_t launch_partition(int mode, const int32_t* flag, const int32_t* alive,
                            const int32_t* fallback, int64_t n, int32_t* counts, int32_t* offsets,
                            int32_t* perm, hipStream_t s);
hipError_t launch_polarization_partials(const double* spin, const int32_t* alive, int64_t n,
                                        double* partials, hipStream_t s);

hipError_t launch_reduce_polarization(const double* partials, int n_blocks, int n_reports,
                                      double* out, hipStream_t stream);

}  // namespace st
