// gfx950 decode kernel of 128-head MLA models (decode_mla.h).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "decode_mla.h"
#include "kargs.h"
#include "schedule.h"

namespace cp {

// 128-head MLA: one workgroup of eight waves per CU.
__global__ __launch_bounds__(64 * MlaCfg::NW, 1) void decode_mla_kernel(const DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) char lds[MlaCfg::LDS];
  __shared__ uint32_t next;
  decode_loop(a, &next, [&](const DecReq &rq, const Seg &sg) { mla_unit(a, a.geom[sg.model], rq, sg, lds); });
}

// ev0 / ev1 (may be null) take the start and end time of the launch.
hipError_t launch_decode_mla(const DecodeArgs &a, int grid, int variant, hipStream_t stream, hipEvent_t ev0,
                              hipEvent_t ev1) {
  const dim3 g(grid);
  switch (variant) {
    case kM_MLA_G128:
      hipExtLaunchKernelGGL(decode_mla_kernel, g, dim3(64 * MlaCfg::NW), 0, stream, ev0, ev1, 0, a);
      return hipGetLastError();
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace cp
