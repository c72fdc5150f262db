// K5 - audit reduce (App. B.2 row-indexed route counters; G1 zero private execution
// under deny): one workgroup of 16 waves (audit_block.h).
#include "audit_block.h"

namespace pmpe {
namespace {

constexpr int AU_WAVES = 16;

__global__ __launch_bounds__(64 * AU_WAVES) void audit_kernel(AuditArgs a) { audit_block<AU_WAVES>(a); }

}  // namespace

hipError_t launch_audit(const AuditArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(audit_kernel, dim3(1), dim3(64 * AU_WAVES), 0, s, a);
  return hipGetLastError();
}

}  // namespace pmpe
