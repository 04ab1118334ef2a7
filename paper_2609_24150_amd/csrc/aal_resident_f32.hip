// Register-resident EAL and WTV losses: the instances for fp32 logits (the
// kernel is in aal_resident_loss.h).
#include "aal_resident_loss.h"

namespace aal {

hipError_t launch_resident_f32(const LossArgs& a, bool* used) { return launch_in<F32>(a, used); }

}  // namespace aal
