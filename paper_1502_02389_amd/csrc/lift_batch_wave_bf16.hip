// The batched form's wavefront kernel for BF16 storage (lift_batch_wave.hpp).
#include "lift_batch_wave.hpp"

namespace lift {

const void *batch_wave_bf16(int acc, bool stamped) { return pick_batch_wave<BF16>(acc, stamped); }

}  // namespace lift
