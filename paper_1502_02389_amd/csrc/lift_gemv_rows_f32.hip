// gemv kernels for rows of any alignment, F32 storage of A (instantiations
// of lift_gemv_rows.hpp).
#include "lift_gemv_rows.hpp"

namespace lift {

const void *gemv_rows_kernel_f32(int acc, int vec_bytes, int lanes, int v, int r)
{
    return pick_gemv_rows<F32>(acc, vec_bytes, lanes, v, r);
}

const void *gemv_rows_wg_kernel_f32(int acc, int v) { return pick_gemv_rows_wg<F32>(acc, v); }

const void *gemv_panel_kernel_f32(int acc, int r) { return pick_gemv_panel<F32>(acc, r); }

}  // namespace lift
