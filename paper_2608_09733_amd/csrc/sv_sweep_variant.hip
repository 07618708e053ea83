// One tile-sweep instantiation per translation unit, selected on the command
// line (-DSVI_VT=double -DSVI_VM=13 -DSVI_VR=5 -DSVI_VNS=1; one entry of
// SVI_VARIANTS), so the variants compile in parallel.
#include <hip/hip_runtime.h>

#include "sv_device.h"
#include "sv_launch.h"
#include "sv_variants.h"

#if !defined(SVI_VT) || !defined(SVI_VM) || !defined(SVI_VR) || !defined(SVI_VNS)
#error "compile with -DSVI_VT= -DSVI_VM= -DSVI_VR= -DSVI_VNS="
#endif

namespace {
template <typename T, int M, int R, int NS>
hipError_t launch_ops(const SweepArgs &a, int grid, hipStream_t s) {
  if constexpr (!svi_has_ops(sizeof(T) == 8, R, NS)) {
    return hipErrorInvalidValue;
  } else {
    hipLaunchKernelGGL((svk::k_sweep<T, M, R, NS>), dim3(grid), dim3(1 << (M - R)), 0, s, a);
    return hipGetLastError();
  }
}

template <typename T, int M, int R, int NS>
int occupancy_ops() {
  int nb = 0;
  if constexpr (svi_has_ops(sizeof(T) == 8, R, NS))
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, svk::k_sweep<T, M, R, NS>, 1 << (M - R), 0) !=
        hipSuccess)
      return 1;
  return nb > 0 ? nb : 1;
}
}  // namespace

hipError_t SVI_VNAME(launch, SVI_VT, SVI_VM, SVI_VR, SVI_VNS)(const SweepArgs &a, int grid,
                                                              hipStream_t s) {
  return launch_ops<SVI_VT, SVI_VM, SVI_VR, SVI_VNS>(a, grid, s);
}

int SVI_VNAME(occ, SVI_VT, SVI_VM, SVI_VR, SVI_VNS)() {
  return occupancy_ops<SVI_VT, SVI_VM, SVI_VR, SVI_VNS>();
}

#if SVI_VNS != 1
hipError_t SVI_VNAME(launchk, SVI_VT, SVI_VM, SVI_VR, SVI_VNS)(const SweepArgs &a, int grid,
                                                               hipStream_t s) {
  hipLaunchKernelGGL((svk::k_sweep_kron2<SVI_VT, SVI_VM, SVI_VR>), dim3(grid),
                     dim3(1 << (SVI_VM - SVI_VR)), 0, s, a);
  return hipGetLastError();
}

int SVI_VNAME(occk, SVI_VT, SVI_VM, SVI_VR, SVI_VNS)() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &nb, svk::k_sweep_kron2<SVI_VT, SVI_VM, SVI_VR>, 1 << (SVI_VM - SVI_VR), 0) != hipSuccess)
    return 1;
  return nb > 0 ? nb : 1;
}
#else
#if (SVI_VM == 13 || SVI_VM == 12) && SVI_VR == 3
#if SVI_VM == 13
hipError_t svk_launch_sweep_dense13(const SweepArgs &a, int grid, hipStream_t s) {
#else
hipError_t svk_launch_sweep_dense12(const SweepArgs &a, int grid, hipStream_t s) {
#endif
  hipLaunchKernelGGL((svk::k_sweep_kron<SVI_VT, SVI_VM, SVI_VR, true>), dim3(grid),
                     dim3(1 << (SVI_VM - SVI_VR)), 0, s, a);
  return hipGetLastError();
}
#endif

hipError_t SVI_VNAME(launchk, SVI_VT, SVI_VM, SVI_VR, SVI_VNS)(const SweepArgs &a, int grid,
                                                               hipStream_t s) {
  hipLaunchKernelGGL((svk::k_sweep_kron<SVI_VT, SVI_VM, SVI_VR>), dim3(grid),
                     dim3(1 << (SVI_VM - SVI_VR)), 0, s, a);
  return hipGetLastError();
}

int SVI_VNAME(occk, SVI_VT, SVI_VM, SVI_VR, SVI_VNS)() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &nb, svk::k_sweep_kron<SVI_VT, SVI_VM, SVI_VR>, 1 << (SVI_VM - SVI_VR), 0) != hipSuccess)
    return 1;
  return nb > 0 ? nb : 1;
}
#endif
