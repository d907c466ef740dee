// Tracking in double precision, the network turns' orbits, and the choice of a kernel
// for a launch (the mixed, extended and team kernels are in files of their own, which
// compile side by side).
#include "track_body.h"

namespace st {

namespace {

// Deterministic second pass of the polarization reduction: one block per
// report sums the per-block partials in a fixed order.
__global__ void __launch_bounds__(256) reduce_polarization_kernel(const double* partials,
                                                                  int n_blocks, double* out) {
  __shared__ double acc[256][4];
  const int rep = blockIdx.x;
  double s[4] = {0, 0, 0, 0};
  for (int b = threadIdx.x; b < n_blocks; b += 256)
    for (int c = 0; c < 4; ++c) s[c] += partials[((int64_t)rep * n_blocks + b) * 4 + c];
  for (int c = 0; c < 4; ++c) acc[threadIdx.x][c] = s[c];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int c = 0; c < 4; ++c) acc[threadIdx.x][c] += acc[threadIdx.x + w][c];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double nal = acc[0][3];
    const double inv = nal > 0 ? 1.0 / nal : 0.0;
    out[rep * 4 + 0] = acc[0][0] * inv;
    out[rep * 4 + 1] = acc[0][1] * inv;
    out[rep * 4 + 2] = acc[0][2] * inv;
    out[rep * 4 + 3] = nal;
  }
}

}  // namespace

int track_block_size() { return kBlock; }

// in the other files
hipError_t launch_mixed(const TrackArgs& a, int nt, hipStream_t stream);
hipError_t launch_ext(const TrackArgs& a, int nt, hipStream_t stream);
hipError_t launch_ext_orbit(const TrackArgs& a, int nt, hipStream_t stream);
hipError_t launch_plain_team(const TrackArgs& a, int nt, hipStream_t stream);
hipError_t launch_ext_team(const TrackArgs& a, int nt, hipStream_t stream);
hipError_t launch_beside(const TrackArgs& fallback, const TrackArgs& orbit, int nt, hipStream_t stream);

hipError_t launch_orbit(const TrackArgs& a, int nt, bool ext, hipStream_t stream) {
  if (ext) return launch_ext_orbit(a, nt, stream);
  const dim3 grid((unsigned)((a.n_lanes + kBlock - 1) / kBlock)), block(kBlock);
  hipLaunchKernelGGL((orbit_kernel<5, false>), grid, block, 0, stream, a);   // no rotation is formed
  return hipGetLastError();
}

hipError_t launch_surrogate_turns(TrackArgs orbit, TrackArgs fallback, const TrackPlan& plan,
                                  hipStream_t stream) {
  if (!plan.team || plan.ext || orbit.n_lanes > kBesideLanes || orbit.n_lanes <= 0 || fallback.n_lanes <= 0) {
    hipError_t e = hipSuccess;
    if (orbit.n_lanes > 0) e = launch_orbit(orbit, plan.nt, plan.ext, stream);
    if (e == hipSuccess && fallback.n_lanes > 0) e = launch_track(fallback, plan, stream);
    return e;
  }
  const int team = team_size();
  fallback.n_blocks = (int32_t)((fallback.n_lanes + team - 1) / team);
  orbit.n_blocks = (int32_t)((orbit.n_lanes + kBlock - 1) / kBlock);
  return launch_beside(fallback, orbit, plan.nt, stream);
}

hipError_t launch_track(TrackArgs a, const TrackPlan& plan, hipStream_t stream) {
  const int per = plan.team ? team_size() : kBlock;
  a.n_blocks = (int32_t)((a.n_lanes + per - 1) / per);
  // the extended methods run in double precision only
  if (plan.ext)
    return plan.team ? launch_ext_team(a, plan.nt, stream) : launch_ext(a, plan.nt, stream);
  if (plan.mixed) return launch_mixed(a, plan.nt, stream);
  return plan.team ? launch_plain_team(a, plan.nt, stream) : launch_nt<false, false>(a, plan.nt, stream);
}

hipError_t launch_reduce_polarization(const double* partials, int n_blocks, int n_reports,
                                      double* out, hipStream_t stream) {
  if (n_reports <= 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_polarization_kernel, dim3(n_reports), dim3(256), 0, stream, partials,
                     n_blocks, out);
  return hipGetLastError();
}

}  // namespace st
