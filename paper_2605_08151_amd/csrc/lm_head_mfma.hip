// Dispatch of the large-tile LM head (lm_head_mfma_kernel.h): row groups, nontemporal stores and loads, instantiation.
#include "lm_head_mfma_kernel.h"

namespace specv {

Tunable g_lm_packed_tile{0};   // benchmark hook: 0 = automatic (this kernel for M > 160 and by lm_packed_large_tile from 113 on), 1 = the weight-streaming kernel over row groups
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

static MfmaLoads mfma_loads(int groups, int H, int V) { return mfma_loads_for(groups, H, V, kMemorySideCache); }

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
    if (g_lm_mfma_rows == 0 && g_lm_mfma_nt == 0) {      // (the benchmark hooks speak of groups of at most 16 tiles)
        const MfmaLayout T = mfma_tall_layout_for(M, V, device_cu_count());
        if (T.groups > 0 && mfma_tall_pays(T, H)) return lm_head_tile(mfma_loads(T.groups, H, V), nt, a, wp, c, M, H, V, T, s);
    }
    switch (mfma_loads(L.groups, H, V)) {
        case kStreamLoads: return L.tm < 11 ? lm_head_tile(kStreamLoads, nt, a, wp, c, M, H, V, L, s) : lm_head_mfma_stream(nt, a, wp, c, M, H, V, L, sm, s);
        case kGlobalLoads: return lm_head_mfma_global(nt, a, wp, c, M, H, V, L, sm, s);
        default: return L.tm < 9 ? lm_head_tile(kBufferLoads, nt, a, wp, c, M, H, V, L, s) : lm_head_mfma_buffer(nt, a, wp, c, M, H, V, L, sm, s);
    }
}

int lm_head_rowmajor(bool stream, bool nt, const uint16_t* a, const uint16_t* w, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s);

// The same on a row-major matrix, for spec_lm_head.  Returns false if it does not take the shape, or other kernels are ahead (see lm_rowmajor_large_tile).
bool lm_head_rowmajor_dispatch(const uint16_t* a, const uint16_t* w, float* c, int M, int H, int V, hipStream_t s, int* rc)
{
    static_assert(kMfRing * kMfSlab == 256, "the rule's multiple of H");
    if (M <= 112 || !lm_rowmajor_large_tile(M, H, V, device_cu_count(), kMemorySideCache)) return false;    // (rows first: the number of CUs is a call into the runtime)
    const MfmaLayout L = mfma_layout_for(M, V, device_cu_count(), 0);
    *rc = lm_head_rowmajor(mfma_loads(L.groups, H, V) == kStreamLoads, M <= 416 && V % 16 == 0, a, w, c, M, H, V, L, s);
    return true;
}

}  // namespace specv
