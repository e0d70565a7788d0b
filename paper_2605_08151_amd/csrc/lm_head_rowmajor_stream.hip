// The large-tile LM head on a row-major vocabulary matrix: nontemporal loads (one row group).
#include "lm_head_mfma_kernel.h"

namespace specv {

int lm_head_rowmajor_stream(bool nt, const uint16_t* a, const uint16_t* w, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s)
{
    return nt ? launch_rowmajor<8, kRowStreamLoads, true>(a, w, c, M, H, V, L, s) : launch_rowmajor<8, kRowStreamLoads, false>(a, w, c, M, H, V, L, s);
}

}  // namespace specv
