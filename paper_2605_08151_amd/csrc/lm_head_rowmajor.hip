// The large-tile LM head on a row-major vocabulary matrix, for spec_lm_head: ordinary loads.
#include "lm_head_mfma_kernel.h"

namespace specv {

int lm_head_rowmajor_stream(bool nt, const uint16_t* a, const uint16_t* w, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s);

int lm_head_rowmajor(bool stream, bool nt, const uint16_t* a, const uint16_t* w, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s)
{
    if (stream) return lm_head_rowmajor_stream(nt, a, w, c, M, H, V, L, s);
    return nt ? launch_rowmajor<8, kRowLoads, true>(a, w, c, M, H, V, L, s) : launch_rowmajor<8, kRowLoads, false>(a, w, c, M, H, V, L, s);
}

}  // namespace specv
