// Stand-ins for the kernel launchers (launch.h) in the host-only sanitizer
// build: the driver exercises the host code of api.hip and control.hip, and
// nothing reaches a launcher there except through paths that need a device.
#include <hip/hip_runtime_api.h>

#include <algorithm>

#include "launch.h"

// With stub_resident > 0 the decode plan sees a device that holds that many
// workgroups of the native kernel (twice as many of the elastic one), and a
// decode launch only records its arguments.
int stub_resident = 0;
ekv::DecodeArgs stub_decode{};

namespace ekv {
hipError_t launch_decode(const DecodeArgs& a, int, int, bool, hipStream_t) {
  stub_decode = a;
  return stub_resident ? hipSuccess : hipErrorNoDevice;
}
hipError_t decode_grid(const DecodeArgs& a, int, int, bool elastic, int* grid) {
  if (!stub_resident) return hipErrorNoDevice;
  const long long wanted = (a.pairs_max + a.min_chunk - 1) / a.min_chunk;
  *grid = (int)std::max<long long>(1, std::min<long long>(std::min(stub_resident * (elastic ? 2 : 1), kMaxDecodeGrid), wanted));
  return hipSuccess;
}
hipError_t launch_zero_u32(uint32_t*, size_t, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_demote(const TransitionArgs&, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_refine(const TransitionArgs&, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_stage(const StageArgs&, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_append(const AppendArgs&, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_prefill(const PrefillArgs&, int, int, bool, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_validate_batch(const ValidateBatchArgs&, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_validate_list(const ValidateListArgs&, hipStream_t) { return hipErrorNoDevice; }
}  // namespace ekv
