// Register-resident EAL and WTV losses: the instances for bf16 logits and the
// dispatch over the logit types (the kernel is in aal_resident_loss.h).
#include "aal_resident_loss.h"

namespace aal {

hipError_t launch_resident(const LossArgs& a, bool* used) {
  *used = false;
  const int E = a.in == DType::kBf16 ? Bf16::kVec : F32::kVec;
  if (a.V % E != 0) return hipSuccess;
  return a.in == DType::kBf16 ? launch_in<Bf16>(a, used) : launch_resident_f32(a, used);
}

}  // namespace aal
