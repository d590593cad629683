// FP32 wave-group step kernels of one number of angle groups per wave
// (RT_NG, given by the build): one translation unit each, so that the build
// compiles the instances in parallel.
#include "rt_internal.hpp"
#include "rt_step3.hpp"

#define RT_CAT2(a, b) a##b
#define RT_CAT(a, b) RT_CAT2(a, b)

namespace rtk {

namespace {

template <bool FUSED, bool SO>
void step3_launch(const StepArgs &a, const KShape &k, long long blocks, hipStream_t s) {
  dim3 g((unsigned)blocks), b(64 * k.waves);
  const size_t lds = step3_lds_bytes(k.waves, (int)sizeof(float));
  if (k.periodic)
    hipLaunchKernelGGL((k_step3<float, float, kAnglesPerWave, RT_NG, true, FUSED, SO>), g, b, lds,
                       s, a);
  else
    hipLaunchKernelGGL((k_step3<float, float, kAnglesPerWave, RT_NG, false, FUSED, SO>), g, b, lds,
                       s, a);
}

struct PackedLaunch {
  dim3 grid, block;
  size_t lds;
  const PackedJob *jobs;
  int waves, team_lds;
  bool periodic;
};

template <int WAVES>
void packed_launch(const PackedLaunch &l, hipStream_t s) {
  if (l.periodic)
    hipLaunchKernelGGL((k_step3_packed<float, float, kAnglesPerWave, RT_NG, true, WAVES>), l.grid,
                       l.block, l.lds, s, l.jobs, l.waves, l.team_lds);
  else
    hipLaunchKernelGGL((k_step3_packed<float, float, kAnglesPerWave, RT_NG, false, WAVES>), l.grid,
                       l.block, l.lds, s, l.jobs, l.waves, l.team_lds);
}

}  // namespace

void RT_CAT(launch_step3_f32_, RT_NG)(const StepArgs &a, const KShape &k, bool fused,
                                      long long blocks, hipStream_t s) {
  if (fused && k.second)
    step3_launch<true, true>(a, k, blocks, s);  // second-order absorption
  else if (fused)
    step3_launch<true, false>(a, k, blocks, s);
  else
    step3_launch<false, false>(a, k, blocks, s);
}

void RT_CAT(launch_packed_f32_, RT_NG)(const PackedJob *jobs, int njobs, int waves, int tiles,
                                       bool periodic, hipStream_t s) {
  // as many teams of `waves` waves as the largest solve has tiles for, within
  // the workgroup's waves and a CU's LDS (21 KB and more a team)
  const size_t lds = step3_lds_bytes(waves, (int)sizeof(float));
  int teams = packed_waves(RT_NG) / waves;
  const int fit = (int)(kLdsPerCu / lds);
  if (teams > fit) teams = fit;
  if (teams > tiles) teams = tiles;
  if (teams < 1) teams = 1;
  const PackedLaunch l{dim3((unsigned)njobs), dim3(64 * waves * teams), lds * teams, jobs, waves,
                       (int)(lds / sizeof(double)), periodic};
  if (waves * teams <= kMaxWaves)
    packed_launch<kMaxWaves>(l, s);
  else
    packed_launch<packed_waves(RT_NG)>(l, s);
}

}  // namespace rtk
