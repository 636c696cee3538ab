// The batched form's wavefront kernel for F32 storage (lift_batch_wave.hpp).
#include "lift_batch_wave.hpp"

namespace lift {

const void *batch_wave_f32(int acc, bool stamped) { return pick_batch_wave<F32>(acc, stamped); }

}  // namespace lift
