// Step launches with FP32 intensities: the wave-group kernels by number of
// angle groups per wave, and the thread-per-cell kernel for more directions
// than they hold, for second-order steps from a given increment and for planes
// of more than 4 GiB.
#include "rt_cellwise.hpp"
#include "rt_internal.hpp"

namespace rtk {

namespace {

template <bool FUSED>
void cell_launch(const StepArgs &a, const KShape &k, long long blocks, hipStream_t s) {
  dim3 g((unsigned)blocks), b(kBlock);
  if (k.second) {
    if (k.periodic)
      hipLaunchKernelGGL((k_step<float, float, true, FUSED, true>), g, b, 0, s, a);
    else
      hipLaunchKernelGGL((k_step<float, float, false, FUSED, true>), g, b, 0, s, a);
  } else if (k.periodic) {
    hipLaunchKernelGGL((k_step<float, float, true, FUSED, false>), g, b, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_step<float, float, false, FUSED, false>), g, b, 0, s, a);
  }
}

}  // namespace

hipError_t launch_step_f32(const StepArgs &a, const KShape &k, bool fused, long long blocks,
                           hipStream_t s) {
  (void)hipGetLastError();  // the result below reports this launch only
  if (k.waves && (fused || !k.second)) {
    switch (k.groups) {
      case 1: launch_step3_f32_1(a, k, fused, blocks, s); break;
      case 2: launch_step3_f32_2(a, k, fused, blocks, s); break;
      case 3: launch_step3_f32_3(a, k, fused, blocks, s); break;
      default: launch_step3_f32_4(a, k, fused, blocks, s); break;
    }
  } else if (fused) {
    cell_launch<true>(a, k, blocks, s);
  } else {
    cell_launch<false>(a, k, blocks, s);
  }
  return hipGetLastError();
}

hipError_t launch_packed_f32(const PackedJob *jobs, int njobs, int waves, int groups,
                             int tiles, bool periodic, hipStream_t s) {
  if (njobs <= 0) return hipSuccess;
  if (waves < 1 || waves > kMaxWaves) return hipErrorInvalidValue;
  (void)hipGetLastError();  // the result below reports this launch only
  switch (groups) {
    case 1: launch_packed_f32_1(jobs, njobs, waves, tiles, periodic, s); break;
    case 2: launch_packed_f32_2(jobs, njobs, waves, tiles, periodic, s); break;
    case 3: launch_packed_f32_3(jobs, njobs, waves, tiles, periodic, s); break;
    case 4: launch_packed_f32_4(jobs, njobs, waves, tiles, periodic, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace rtk
