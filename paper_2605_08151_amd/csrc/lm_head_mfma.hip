// Dispatch of the large-tile LM head (lm_head_mfma_kernel.h): row groups, nontemporal stores and loads, instantiation.
#include "lm_head_mfma_kernel.h"

namespace specv {

Tunable g_lm_packed_tile{0};   // benchmark hook: 0 = automatic (this kernel for M > 160), 1 = the weight-streaming kernel over row groups
Tunable g_lm_mfma_nt{0};       // benchmark hook: nontemporal logits stores, 0 = automatic (see mfma_nt), 1 = always, 2 = never
Tunable g_lm_mfma_rows{0};     // benchmark hook: rows per group of this kernel at most (144..256), 0 = automatic (256)

static MfmaLayout mfma_layout(int M, int V) { return mfma_layout_for(M, V, device_cu_count(), g_lm_mfma_rows); }

// Nontemporal stores of the logits: nobody reads them before the next kernel, and they do not push the weight stream out of the caches.  Up to 416
// rows, where that stream bounds the kernel (ordinary -> nontemporal, V = 151936, H = 4096: M = 192 294 -> 270 us, M = 257 370 -> 358,
// M = 416 448 -> 450; M = 512 519 -> 522), and only where every row starts on a multiple of 64 bytes: elsewhere rows share their first and
// last lines with their neighbours, and such lines are written to HBM in parts (H = 1280, M = 320: V = 50020 48 -> 56 us, V = 50021 48 -> 57;
// V = 50016 46.8 -> 47.7).
static bool mfma_nt(int M, int V)
{
    const int forced = g_lm_mfma_nt;
    return forced == 1 || (forced == 0 && M <= 416 && V % 16 == 0);
}

// lm_head_mfma_summary.hip (the instantiations that also leave block summaries, built beside these)
int lm_head_mfma_summary(bool nt, const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, const LmSummary& sm, hipStream_t s);

// blocks per row of the summaries for this shape; 0 if the large-tile kernel does not take it
int lm_head_mfma_blocks(int M, int H, int V)
{
    // (V % 4 == 0: the summaries are taken while whole rows of the tile are stored; 32-bit element indices)
    if (M <= 0 || V <= 0 || V % 4 != 0 || H <= 0 || H % (kMfRing * kMfSlab) != 0) return 0;
    const MfmaLayout L = mfma_layout(M, V);
    if ((size_t)M * (size_t)L.blocks >= ((size_t)1 << 32)) return 0;
    return (L.tm >= 9 && L.tm <= 16) ? L.blocks : 0;
}

// Returns SPEC_OK after enqueueing, or a negative status.  summary == nullptr: logits only.
int lm_head_mfma_dispatch(const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const LmSummary* summary, hipStream_t s)
{
    const MfmaLayout L = mfma_layout(M, V);
    if (H % (kMfRing * kMfSlab) != 0)
        return fail(SPEC_ESHAPE, "spec_lm_head_packed: H=%d must be a multiple of %d", H, kMfRing * kMfSlab);
    LmSummary sm{};
    if (summary) {
        if (lm_head_mfma_blocks(M, H, V) == 0)
            return fail(SPEC_ESHAPE, "spec_lm_head_packed_summary: no block summaries for M=%d H=%d V=%d (V must be a multiple of 4)", M, H, V);
        sm = *summary; sm.blocks = L.blocks; sm.passes_per_range = L.passes_per_range;
    }
    const bool nt = mfma_nt(M, V);
    if (summary) return lm_head_mfma_summary(nt, a, wp, c, M, H, V, L, sm, s);
    // One row group reads W once, bound by that stream: nontemporal, by the rule of the weight-streaming kernel (the tree step, M = 188, V = 151936,
    // H = 4096 378 -> 360 us, M = 216 408 -> 394; V = 64000, H = 2560 179 -> 167).
    const bool stream = L.groups == 1 && (size_t)V * H * 2 > kMemorySideCache * 3 / 8;
    switch (L.tm) {
#define SPECV_MF(TMv)                                                                                             \
        case TMv:                                                                                                 \
            return nt ? launch_mfma<TMv, false, true, false>(a, wp, c, M, H, V, L, sm, s)                         \
                      : launch_mfma<TMv, false, false, false>(a, wp, c, M, H, V, L, sm, s);
#define SPECV_MF_ONE_GROUP(TMv)                                                                                   \
        case TMv:                                                                                                 \
            if (stream) return nt ? launch_mfma<TMv, true, true, false>(a, wp, c, M, H, V, L, sm, s)              \
                                  : launch_mfma<TMv, true, false, false>(a, wp, c, M, H, V, L, sm, s);            \
            return nt ? launch_mfma<TMv, false, true, false>(a, wp, c, M, H, V, L, sm, s)                         \
                      : launch_mfma<TMv, false, false, false>(a, wp, c, M, H, V, L, sm, s);
        SPECV_MF(9) SPECV_MF(10)                      // (more than 160 rows in one group: 11 tiles or more)
        SPECV_MF_ONE_GROUP(11) SPECV_MF_ONE_GROUP(12) SPECV_MF_ONE_GROUP(13) SPECV_MF_ONE_GROUP(14) SPECV_MF_ONE_GROUP(15) SPECV_MF_ONE_GROUP(16)
#undef SPECV_MF
#undef SPECV_MF_ONE_GROUP
        default: break;
    }
    return fail(SPEC_ESHAPE, "spec_lm_head_packed: no large-tile instantiation for %d row tiles per group", L.tm);
}

}  // namespace specv
