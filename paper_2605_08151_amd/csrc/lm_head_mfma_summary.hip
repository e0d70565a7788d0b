// The instantiations of the large-tile LM head that also leave block summaries (LmSummary).
#include "lm_head_mfma_kernel.h"

namespace specv {

SPECV_MFMA_FILE(lm_head_mfma_summary) { return launch_mfma_tiles<kBufferLoads, true, 9>(nt, a, wp, c, M, H, V, L, sm, s); }

}  // namespace specv
