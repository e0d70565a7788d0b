// The instantiations of the large-tile LM head with W by nontemporal loads (one row group: 11 row tiles or more).
#include "lm_head_mfma_kernel.h"

namespace specv {

SPECV_MFMA_FILE(lm_head_mfma_stream) { return launch_mfma_tiles<kStreamLoads, false, 11>(nt, a, wp, c, M, H, V, L, sm, s); }

}  // namespace specv
