// gemv kernels for rows of any alignment, BF16 storage of A (instantiations
// of lift_gemv_rows.hpp).
#include "lift_gemv_rows.hpp"

namespace lift {

const void *gemv_rows_kernel_bf16(int acc, int vec_bytes, int lanes, int v, int r)
{
    return pick_gemv_rows<BF16>(acc, vec_bytes, lanes, v, r);
}

const void *gemv_rows_wg_kernel_bf16(int acc, int v) { return pick_gemv_rows_wg<BF16>(acc, v); }

const void *gemv_panel_kernel_bf16(int acc, int r) { return pick_gemv_panel<BF16>(acc, r); }

}  // namespace lift
