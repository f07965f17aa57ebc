// The backward's matrix stages for head dim 64, long launches (a translation unit per head dim and program: they take the longest to compile).
#include "attn_bwd_matrix.h"

namespace sp {

sp_status launch_attn_bwd_matrix_long_d64(const AttnArgs& a, hipStream_t st) {
    return a.row_lo != nullptr ? launch_matrix<64, true, true>(a, st) : launch_matrix<64, false, true>(a, st);
}

}  // namespace sp
