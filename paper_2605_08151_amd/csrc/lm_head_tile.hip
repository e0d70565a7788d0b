// The instantiations of the large-tile LM head with 17 and 18 row tiles per group, and those for one group of 113 to 160 rows that lm_head_mfma_buffer.hip lacks.
#include "lm_head_mfma_kernel.h"

namespace specv {

template <MfmaLoads LOADS, bool NT>
static int launch_tile_count(const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s)
{
    if constexpr (LOADS == kStreamLoads) {
        if (L.tm == 9) return launch_tile<9, LOADS, NT>(a, wp, c, M, H, V, L, s);
        if (L.tm == 10) return launch_tile<10, LOADS, NT>(a, wp, c, M, H, V, L, s);
    }
    if constexpr (LOADS != kGlobalLoads) {
        if (L.tm == 8) return launch_tile<8, LOADS, NT>(a, wp, c, M, H, V, L, s);
    }
    return L.tm == 17 ? launch_tile<17, LOADS, NT>(a, wp, c, M, H, V, L, s) : launch_tile<18, LOADS, NT>(a, wp, c, M, H, V, L, s);
}

int lm_head_tile(MfmaLoads loads, bool nt, const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s)
{
    if (!mf_tile_built(loads, L.tm)) return fail(SPEC_ESHAPE, "spec_lm_head_packed: no instantiation for %d row tiles per group", L.tm);
    switch (loads) {
        case kStreamLoads: return nt ? launch_tile_count<kStreamLoads, true>(a, wp, c, M, H, V, L, s) : launch_tile_count<kStreamLoads, false>(a, wp, c, M, H, V, L, s);
        case kGlobalLoads: return launch_tile_count<kGlobalLoads, false>(a, wp, c, M, H, V, L, s);
        default: return nt ? launch_tile_count<kBufferLoads, true>(a, wp, c, M, H, V, L, s) : launch_tile_count<kBufferLoads, false>(a, wp, c, M, H, V, L, s);
    }
}

}  // namespace specv
