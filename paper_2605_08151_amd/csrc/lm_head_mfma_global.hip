// The instantiations of the large-tile LM head with W by global loads.
#include "lm_head_mfma_kernel.h"

namespace specv {

SPECV_MFMA_FILE(lm_head_mfma_global) { return launch_mfma_tiles<kGlobalLoads, false, 9>(nt, a, wp, c, M, H, V, L, sm, s); }

}  // namespace specv
