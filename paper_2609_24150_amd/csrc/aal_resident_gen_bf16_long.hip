// Register-resident schedule of the combined objectives: the instances for
// bf16 logits with a bf16 gradient and K of 9 to 16 (the kernel is in aal_resident_gen.h;
// the instances are spread over files so that they build in parallel).
#include "aal_resident_gen.h"

namespace aal {

hipError_t launch_general_resident_bf16_long(const GenArgs& a, bool* used) { return launch_tg<Bf16, GBf16, 9>(a, used); }

}  // namespace aal
