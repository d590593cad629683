// Step launches with FP64 intensities: the wave-group kernels by number of
// angles per wave, and the thread-per-cell kernel for second-order steps from
// a given increment or with more directions than a block's waves hold, and for
// planes of more than 4 GiB.  No packed persistent kernel: the serving runtime
// runs FP64 requests through the per-step launches.
#include "rt_cellwise.hpp"
#include "rt_internal.hpp"

namespace rtk {

namespace {

template <bool FUSED>
void cell_launch(const StepArgs &a, const KShape &k, long long blocks, hipStream_t s) {
  dim3 g((unsigned)blocks), b(kBlock);
  if (k.second) {
    if (k.periodic)
      hipLaunchKernelGGL((k_step<double, double, true, FUSED, true>), g, b, 0, s, a);
    else
      hipLaunchKernelGGL((k_step<double, double, false, FUSED, true>), g, b, 0, s, a);
  } else if (k.periodic) {
    hipLaunchKernelGGL((k_step<double, double, true, FUSED, false>), g, b, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_step<double, double, false, FUSED, false>), g, b, 0, s, a);
  }
}

}  // namespace

void launch_step64(const StepArgs &a, const KShape &k, Launch64 what, long long blocks,
                   hipStream_t s) {
  switch (k.geo.slots) {
#define RT_CASE(ns) \
  case ns: launch_step64_##ns(a, k, what, blocks, s); break;
    RT_SLOTS64(RT_CASE)
#undef RT_CASE
  }
}

hipError_t launch_step_f64(const StepArgs &a, const KShape &k, bool fused, long long blocks,
                           hipStream_t s) {
  (void)hipGetLastError();  // the result below reports this launch only
  if (k.waves && (fused || !k.second)) {
    launch_step64(a, k, fused ? kStep64 : kSourceStep64, blocks, s);
  } else if (fused) {
    cell_launch<true>(a, k, blocks, s);
  } else {
    cell_launch<false>(a, k, blocks, s);
  }
  return hipGetLastError();
}

}  // namespace rtk
