// Teams on plain lattices, and surrogate turns beside them.
#include "team_body.h"

namespace st {

namespace {

// Surrogate tracking, the turns between two audits: the fallback particles in
// teams and the orbits of those on the network side by side, on disjoint lanes.
// Each alone is bound by its chain, not by the chip: nine turns of 52000 orbits and
// 13600 fallback particles took 6.0 and 7.6 ms one after the other.  65536
// particles over 20 turns: 48.0 -> 38.5 ms with the teams taking all of them.
template <int NT>
__global__ void __launch_bounds__(kTeam * kTeamWaves) __attribute__((amdgpu_waves_per_eu(2)))
surrogate_kernel(const TrackArgs fallback, const TrackArgs orbit) {
  static_assert(kTeam * kTeamWaves == kBlock);
  __shared__ union {
    TeamShared team;
    BlockShared block;
  } sh;
  const int block = blockIdx.x;
  if (block < fallback.n_blocks)
    team_body<NT, false>(fallback, block, sh.team);
  else
    track_body<5, false, false, true>(orbit, block - fallback.n_blocks, sh.block);
}

}  // namespace

int team_size() { return kTeam; }

hipError_t launch_plain_team(const TrackArgs& a, int nt, hipStream_t stream) {
  return launch_team<false>(a, nt, stream);
}

hipError_t launch_beside(const TrackArgs& fallback, const TrackArgs& orbit, int nt,
                         hipStream_t stream) {
  const dim3 grid((unsigned)(fallback.n_blocks + orbit.n_blocks)), block(kBlock);
  switch (nt) {
    case 5:  hipLaunchKernelGGL(surrogate_kernel<5>, grid, block, 0, stream, fallback, orbit); break;
    case 6:  hipLaunchKernelGGL(surrogate_kernel<6>, grid, block, 0, stream, fallback, orbit); break;
    case 8:  hipLaunchKernelGGL(surrogate_kernel<8>, grid, block, 0, stream, fallback, orbit); break;
    case 9:  hipLaunchKernelGGL(surrogate_kernel<9>, grid, block, 0, stream, fallback, orbit); break;
    case 12: hipLaunchKernelGGL(surrogate_kernel<12>, grid, block, 0, stream, fallback, orbit); break;
    default: hipLaunchKernelGGL(surrogate_kernel<16>, grid, block, 0, stream, fallback, orbit); break;
  }
  return hipGetLastError();
}

}  // namespace st
