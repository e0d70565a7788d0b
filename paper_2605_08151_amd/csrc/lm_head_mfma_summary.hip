// The instantiations of the large-tile LM head that also leave block summaries (LmSummary).
#include "lm_head_mfma_kernel.h"

namespace specv {

int lm_head_mfma_summary(bool nt, const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, const LmSummary& sm, hipStream_t s)
{
    switch (L.tm) {
#define SPECV_MF(TMv)                                                                                             \
        case TMv:                                                                                                 \
            return nt ? launch_mfma<TMv, false, true, true>(a, wp, c, M, H, V, L, sm, s)                          \
                      : launch_mfma<TMv, false, false, true>(a, wp, c, M, H, V, L, sm, s);
        SPECV_MF(9) SPECV_MF(10) SPECV_MF(11) SPECV_MF(12) SPECV_MF(13) SPECV_MF(14) SPECV_MF(15) SPECV_MF(16)
#undef SPECV_MF
        default: break;
    }
    return fail(SPEC_ESHAPE, "spec_lm_head_packed_summary: no large-tile instantiation for %d row tiles per group", L.tm);
}

}  // namespace specv
