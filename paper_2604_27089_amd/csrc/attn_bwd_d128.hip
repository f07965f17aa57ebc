// The backward's matrix stages for head dim 128 (a translation unit per head dim and program: they take the longest to compile).
#include "attn_bwd_matrix.h"

namespace sp {

sp_status launch_attn_bwd_matrix_d128(const AttnArgs& a, hipStream_t st) {
    return a.row_lo != nullptr ? launch_matrix<128, true, false>(a, st) : launch_matrix<128, false, false>(a, st);
}

}  // namespace sp
