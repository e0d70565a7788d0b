// spec_lm_head_packed for batches of more than 160 rows, and for 113 to 160 where it is ahead of the weight-streaming kernel: the MFMA-bound kernel (paper, Appendix "Target side": every
// position of every verification candidate is scored; the hybrid ordinary-parallel batch has ~1200 positions).
//
// With hundreds of rows the LM head is a dense contraction bound by the matrix cores, and what starves them is operand
// traffic: L2 -> CU bytes per flop fall with the workgroup's tile area, LDS bytes per flop with the vocabulary width a wave
// covers.  So: ONE wave per SIMD with the whole register file (512 registers), each wave holding a tile of
// 16 TM rows x 64 vocabulary entries in the accumulation registers (TM <= 16: the workgroup tile is up to 256 x 256; 17 and 18 with the rest
// in vector registers),
//   * W goes from L2/HBM straight into MFMA operand registers (the packed layout is the A operand of
//     v_mfma_f32_16x16x32_bf16 lane by lane), through a ring of 4 slabs of 64 k, each chunk requested again right
//     after the MFMAs that consumed it: no W byte touches LDS;
//   * hidden goes from L2 into LDS by direct global->LDS loads (no staging registers), 4 slabs of 64 k deep, and
//     a fragment read from LDS feeds 4 MFMAs (one per panel of the wave);
//   * a wave is its own latency hiding: everything it needs is requested 2.5 to 4 slabs (2-4 us) ahead, hidden fragments are read
//     from LDS across the border of two slabs, and the stores of a tile drain under the first steps of the next one.
// What bounds it: the issue slots (a wave issues 16 instructions in the time of 4 MFMAs, 64 cycles), and the power that the operands' way from L2
// costs.  M = 1152, V = 151936, H = 4096 takes 1097 us in groups of 18 tiles (1.31 PFLOP/s), 1150 of 15 (1240-1270 with vector address arithmetic, branches
// per group and a full stop at every slab and tile; 1119 without any store of logits, 800 with operands that stay in registers).  With one row group (113..288 rows) it is the stream of W,
// as in the weight-streaming kernel: M = 188 247 us, 5.5 TB/s.
// The batch is cut into row groups of whole 16-row tiles, nearly equal and at most 288 rows each; the grid is groups x panel ranges, the groups of a
// range run on the same XCD at the same time and share that range's panels through the XCD's L2, so HBM sees W once.
// Per output element the products are added in the same order as in the other LM-head kernels (k ascending, one
// fp32 accumulator), so the logits are bit-identical to theirs.
#pragma once

#include "common.h"
#include "lm_head_tiles.h"

#include <type_traits>
#include <utility>

namespace specv {

constexpr int kMfSlab = 64;                    // k per slab
constexpr int kMfPitch = kMfSlab * 2;          // bytes per hidden row in LDS; 16-byte chunk c of row r sits at c ^ ((r >> 1) & 7)
constexpr int kMfRing = 4;                     // slabs in flight: hidden slabs in LDS = W slabs in registers
// bytes per row of a wave's store patch: padded by 16, or for more than 16 row tiles, which leave no LDS for padding, swizzled
constexpr int mf_patch_pitch(int tm) { return kMfTN * 64 + (tm > 16 ? 0 : 16); }
constexpr size_t mf_lds_bytes(int tm, bool summary)
{
    return (size_t)kMfRing * ((tm * 16 + 31) / 32 * 32) * kMfPitch + (size_t)kMfWaves * 16 * mf_patch_pitch(tm) + (summary ? tm * 16 * 4 : 0);
}

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // (a row of logits starts at any multiple of 4 bytes)

#define SPECV_INLINE __attribute__((always_inline))
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// LOADS: how W is read, see MfmaLoads; NT: nontemporal stores of the logits (a template argument: of two stores in the branches of a flag the compiler makes one ordinary store);
// SUMMARY instantiations also leave the block summaries described at LmSummary.

template <int TM, MfmaLoads LOADS, bool NT, bool SUMMARY>
__device__ __forceinline__ void lm_head_mfma_tiles(
    const uint16_t* __restrict__ A_all, const uint16_t* __restrict__ Wp, float* __restrict__ C_all,
    int M_all, int H, int V, int n_panels, int panels_per_wg, int groups, int tiles_lo, int groups_hi,
    LmSummary sm)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int RW = kMfRing;
    constexpr int SR = (TM * 16 + 31) / 32 * 32;      // rows staged per slab: 8 per direct load, the same count for every wave
    constexpr int QN = SR / 32;                       // direct loads per wave and slab
    constexpr int kSlabBytes = SR * kMfPitch;
    // hidden fragments are read from LDS ahead of their MFMAs: kHfCross groups at the border of two steps, kHfAhead inside one
    constexpr int kHfCross = TM >= 9 ? 5 : 4, kHfAhead = 7, kHfCatchUp = kHfAhead - kHfCross, kHfRing = 8;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, l16 = lane & 15, kg = lane >> 4;
    // Workgroup -> (row group, panel range): workgroups are dealt round-robin to the 8 XCDs, so the groups of one range
    // are given consecutive slots of the same XCD.
    const int xcd = blockIdx.x & 7, dealt = blockIdx.x >> 3;
    const int group = dealt % groups, range = (dealt / groups) * 8 + xcd;
    // Row groups are whole 16-row tiles: the first groups_hi groups have tiles_lo + 1 = TM of them, the others tiles_lo.
    // A group with TM - 1 tiles issues no MFMA for the missing one: on this chip an MFMA that computes nothing still costs
    // the power that sets the clock for all the others.
    const int row0 = 16 * (group * tiles_lo + min(group, groups_hi));
    const bool full_tm = group < groups_hi || tiles_lo == TM;
    const int M = min(16 * (tiles_lo + (group < groups_hi ? 1 : 0)), M_all - row0);    // >= 1 by the host's choice of groups
    const unsigned char* __restrict__ A = reinterpret_cast<const unsigned char*>(A_all + (size_t)row0 * H);
    float* __restrict__ C = C_all + (size_t)row0 * V;
    const int p_begin = range * panels_per_wg;
    const int p_end = min(n_panels, p_begin + panels_per_wg);
    if (p_begin >= p_end) {
        if constexpr (SUMMARY) {                      // a range past the matrix: its block slots hold nothing
            if (group == 0)
                for (int b = tid; b < sm.passes_per_range * kMfWaves; b += 64 * kMfWaves) {
                    sm.blk_span[2 * (range * sm.passes_per_range * kMfWaves + b)] = 0;
                    sm.blk_span[2 * (range * sm.passes_per_range * kMfWaves + b) + 1] = 0;
                }
        }
        return;
    }
    const int n_own = p_end - p_begin;
    const int npass = (n_own + kMfPassPanels - 1) / kMfPassPanels;
    const int nslab = H / kMfSlab;                    // a multiple of 4 (host check)

    unsigned char* hbuf = smem;                                        // kMfRing slabs
    constexpr int kPatchPitch = mf_patch_pitch(TM);
    // position of the 16 bytes that hold entries 4 c .. 4 c + 3 of row r in the wave's store patch
    auto patch_at = [&](int r, int c) SPECV_INLINE {
        if constexpr (kPatchPitch == kMfTN * 64) c ^= r;
        return r * kPatchPitch + c * 16;
    };
    unsigned char* patch = smem + kMfRing * kSlabBytes + wave * (16 * kPatchPitch);
    float* row_scale = reinterpret_cast<float*>(smem + kMfRing * kSlabBytes + kMfWaves * (16 * kPatchPitch));   // [TM * 16], SUMMARY only
    if constexpr (SUMMARY) {
        // log2(e) / T of each row's request (0: greedy, or no such row); read again only after many barriers
        for (int r = tid; r < TM * 16; r += 64 * kMfWaves) {
            float sc = 0.0f;
            if (r < M) {
                int lo = 0, hi = sm.B - 1;                // largest i with qo_indptr[i] <= row
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (sm.qo_indptr[mid] <= row0 + r) lo = mid; else hi = mid - 1;
                }
                const float T = sm.temperature[lo];
                sc = T > 0.0f ? (float)(1.4426950408889634 / (double)T) : 0.0f;
            }
            row_scale[r] = sc;
        }
    }

    // ---- hidden: byte offset (from A) of the 16 bytes this lane moves in direct load q of a slab, k0 = 0.
    // Load q of wave w fills LDS rows 8 (QN w + q) .. +7: lane l writes position l % 8 of row 8 (QN w + q) + l / 8,
    // which must hold chunk (l % 8) ^ ((row >> 1) & 7) of that row.  Rows past the group repeat its last row.
    uint32_t hoff[QN];
#pragma unroll
    for (int q = 0; q < QN; ++q) {
        const int row = 8 * (QN * wave + q) + (lane >> 3);
        const int ch = (lane & 7) ^ ((row >> 1) & 7);
        hoff[q] = (uint32_t)min(row, M - 1) * (uint32_t)H * 2u + (uint32_t)ch * 16u;
    }
    const unsigned char* hsrc = A;                    // slab whose direct loads are issued next (wave-uniform: a scalar base)
    auto stage_h1 = [&](int slot, int q) SPECV_INLINE {            // direct load q of this wave's share of that slab
        lds_dma16_off(hoff[q], hsrc, hbuf + slot * kSlabBytes + (QN * wave + q) * 1024);
    };

    // ---- W: the wave's panels of a pass, read at a scalar position (panel slot and place in the stream) from its first panel on, through a buffer
    // descriptor or by address, plus 16 bytes per lane: a request costs no vector address arithmetic.
    int wave_p0 = 0, wave_np = 0;
    auto pass_panels = [&](int pass, int& p0, int& np) SPECV_INLINE {
        const PanelShare s = mf_panel_share(p_begin, p_end, pass, wave);
        p0 = s.p0;
        np = s.np;
    };
    // Row-major (ROWS): a load takes 128 bytes (a slab) of 8 rows, whole lines.  The two loads of a slab and panel slot, rows 0..7 and 8..15, become the operands
    // of its two k-tiles by selections and a rotation within 16 lanes (weave_rows) when the slab's step begins.
    constexpr bool ROWS = LOADS == kRowLoads || LOADS == kRowStreamLoads;
    const uint32_t panel_bytes = (uint32_t)H * 32u;
    const uint32_t woff = (uint32_t)lane * 16u;
    uint32_t roff[kMfTN][2];                          // (ROWS) byte offset of this lane's 16 bytes from the wave's first row
    u32x4 wreg[RW][2][kMfTN];
    __amdgpu_buffer_rsrc_t wrsrc;
    const unsigned char* wbase = nullptr;
    uint32_t wpos = 0;                                // byte position of the slab that is requested next inside its panel
    uint32_t wslot[kMfTN];                            // mf_slot_bytes of the wave's panel slots
    auto open_panels = [&](int p0, int np) SPECV_INLINE {
        const unsigned char* base = reinterpret_cast<const unsigned char*>(Wp) + (size_t)p0 * panel_bytes;
        if constexpr (LOADS == kBufferLoads) wrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (uint32_t)max(np, 1) * panel_bytes, 0x00020000);
        wbase = base;
        wpos = 0;
#pragma unroll
        for (int tn = 0; tn < kMfTN; ++tn) {
            if constexpr (ROWS) {
                // entries past V repeat the last one; which half of a row's 128 bytes the lane takes: see weave_rows
                const int last = V - 1 - p0 * 16, row = min(tn, max(np - 1, 0)) * 16 + (l16 & 7);
                roff[tn][0] = (uint32_t)min(row, last) * (uint32_t)H * 2u + (uint32_t)(kg + (l16 & 8) / 2) * 16u;
                roff[tn][1] = (uint32_t)min(row + 8, last) * (uint32_t)H * 2u + (uint32_t)(kg + 4 - (l16 & 8) / 2) * 16u;
            } else {
                wslot[tn] = mf_slot_bytes(np, tn, panel_bytes);
            }
        }
    };
    constexpr uint32_t kWSlab = ROWS ? kMfSlab * 2 : 2048;         // bytes from a slab to the next in a row, in a packed panel
    auto fetch_w1 = [&](int slot, int t, int tn) SPECV_INLINE {    // k-tile t of that slab, panel slot tn
        const u32x4* at;
        if constexpr (ROWS) at = reinterpret_cast<const u32x4*>(wbase + wpos + roff[tn][t]);
        else at = reinterpret_cast<const u32x4*>(wbase + (wpos + t * 1024 + wslot[tn]) + woff);
        if constexpr (LOADS == kStreamLoads || LOADS == kRowStreamLoads) wreg[slot][t][tn] = __builtin_nontemporal_load(at);
        else if constexpr (LOADS != kBufferLoads) wreg[slot][t][tn] = *at;
        else wreg[slot][t][tn] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, woff, wpos + t * 1024 + wslot[tn], 0);
    };

    // (ROWS) Loaded, lane (l16, kg) of slot tn holds row l16 % 8, 16-byte piece kg (l16 < 8) or 4 + kg (else), and row 8 + l16 % 8, piece 4 + kg or kg; needed is row
    // l16, pieces kg and 4 + kg: a selection, and a selection and a rotation by 8 within the 16 lanes.
    auto weave_rows = [&](auto rc, auto slots_c) SPECV_INLINE {
        constexpr int r = decltype(rc)::value;
        const bool low = l16 < 8;
#pragma unroll
        for (int tn = 0; tn < decltype(slots_c)::value; ++tn) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t a = wreg[r][0][tn][e], b = wreg[r][1][tn][e];
                wreg[r][0][tn][e] = low ? a : b;
                wreg[r][1][tn][e] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(low ? b : a), 0x128, 0xF, 0xF, false);   // row_ror:8
            }
            asm volatile("" : "+v"(wreg[r][0][tn]), "+v"(wreg[r][1][tn]));
        }
        asm volatile("s_nop 1");                      // (the products are assembly statements)
        __builtin_amdgcn_sched_barrier(0);
    };

    f32x4 acc[kMfTN][TM];
#pragma unroll
    for (int tn = 0; tn < kMfTN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = f32x4{0.f, 0.f, 0.f, 0.f};

    // LDS offset of this lane's fragment of row tile 0, k-tile t inside a slab: row l16, chunk (4 t + kg) ^ ((l16 >> 1) & 7)
    // (row 16 tm + l16 has the same swizzle term: 8 tm vanishes under & 7)
    // and the same for the other slots, so that every fragment is one of four registers (eight where two slabs are too long) plus a 16-bit immediate
    typedef __attribute__((address_space(3))) const unsigned char* LdsPtr;
    constexpr int kHfSlots = kSlabBytes + (TM - 1) * 16 * kMfPitch < 65536 ? 2 : 1;      // ring slots per register
    uint32_t hf_at[RW / kHfSlots][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < RW / kHfSlots; ++u) {
            hf_at[u][t] = (uint32_t)(uintptr_t)(LdsPtr)hbuf + (uint32_t)(u * kHfSlots * kSlabBytes + l16 * kMfPitch + (((t * 4 + kg) ^ ((l16 >> 1) & 7)) << 4));
            asm volatile("" : "+v"(hf_at[u][t]));     // (the compiler would keep a register per distant fragment instead)
        }
    bf16x8 hfq[kHfRing];
    auto hfrag = [&](auto rc, auto ic) SPECV_INLINE {              // fragment i = t * TM + tm of the slab in ring slot r
        constexpr int r = decltype(rc)::value, i = decltype(ic)::value;
        static_assert((kHfSlots - 1) * kSlabBytes + (TM - 1) * 16 * kMfPitch < 65536, "16-bit LDS offsets");
        return *reinterpret_cast<__attribute__((address_space(3))) const bf16x8*>(
            (LdsPtr)(uintptr_t)hf_at[r / kHfSlots][i / TM] + ((r % kHfSlots) * kSlabBytes + (i % TM) * (16 * kMfPitch)));
    };

    int pass = 0, p0_next, np_next;
    pass_panels(0, wave_p0, wave_np);
    pass_panels(npass > 1 ? 1 : 0, p0_next, np_next);
    open_panels(wave_p0, wave_np);
    // prologue: hidden slabs 0..2 and W slabs 0..3 except the last chunk (the first step requests it); everything has landed
    // before the first step (once per workgroup)
#pragma unroll
    for (int r = 0; r < RW - 1; ++r) {
#pragma unroll
        for (int q = 0; q < QN; ++q) stage_h1(r, q);
        hsrc += kMfSlab * 2;
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int tn = 0; tn < kMfTN; ++tn)
                if (r < RW - 1 || t == 0) fetch_w1(r, t, tn);
        if (r < RW - 1) wpos += kWSlab;
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    static_for<kHfCross>([&](auto ic) SPECV_INLINE { hfq[ic] = hfrag(std::integral_constant<int, 0>{}, ic); });
    __builtin_amdgcn_sched_barrier(0);

    // One step = one slab of 64 k for the whole tile; slab s lives in ring slot s % 4 (hidden in LDS, W in registers), and
    // because H is a multiple of 256 that slot is the same in every pass, so all ring indices are compile-time constants.
    // The steps of all passes form one stream: the requests for the slabs after the end of a pass are the first slabs of
    // the next pass, so the pipeline never drains between tiles.
    // A step is 2 TM groups of 4 MFMAs (one hidden fragment against the wave's 4 panels).  A wave issues one instruction in
    // 4 cycles and a group keeps the matrix core busy for 64: everything else of a group has to fit 12 slots, so a request is
    // one load with a scalar base and a step does no vector arithmetic.
    // Requests of step s, in program order (fenced: the in-order completion of a wave's requests is what every wait counts on):
    //   groups 0..3            W chunk k-tile 1 of slab s+3 (its ring slot was consumed at the end of the previous step)
    //   groups 4..4+QN-1       direct loads of hidden slab s+3 into the LDS slot of slab s-1
    //   groups TM..TM+3        W chunk k-tile 0 of slab s+4 (this step's slot, consumed by groups 0..TM-1)
    // Hidden fragments are read 5 to 7 groups ahead, across the border of the steps: the barrier that publishes slab s+1 and
    // frees the slot of slab s stands 5 groups before the end of step s, when this step's last fragment has been in registers
    // for two groups, and the last groups read the first fragments of slab s+1: no step begins by waiting for LDS.
    // The accumulators are pinned to the accumulation registers by writing the MFMA as an asm statement; its operands are
    // ordinary values, so the compiler still inserts the waits for the W loads and the LDS reads.  It does not know that an MFMA must
    // not follow a vector instruction that wrote its operand by less than 2 wait states.  Before the first step of a pass, where copies do stand,
    // the MFMAs bring their own s_nop; that nothing else is in the way, around the branches for the last row tile and for panel slots above all, is
    // checked on the built code by a test (s_nops at those branches too: M = 768, V = 32000, H = 4096 161 -> 164 us, M = 1152 263 -> 279).  Those waits count W
    // loads only (the direct loads are invisible to the compiler): a wait for a chunk allows 7 SLOTS younger requests in flight, of the 2 SLOTS + QN of a step, direct loads
    // among them.  With 4 slots that is 1.75 steps at 8 direct loads a step and 1.65 at 9 (17 and 18 tiles), less than the 2.5 steps a direct load has, which thus is seldom what the math
    // waits for; in a last pass of two panels per wave it is 1.1 to 1.75, and the math does wait for direct loads before they are needed.  That slab s+1 is complete in LDS is not
    // left to this: the counted wait in front of its barrier says so.
    static_assert(4 + QN <= TM && TM + 3 <= 2 * TM - kHfCross - 1, "the requests of a step precede its barrier");
    // FIRST: the first slab of a pass (the products start from zero).  SLOTS: panels per wave whose products are taken.  last_iter: the last 4 slabs of a pass.
    // stores: the counted stores of a tile were issued between the requests for slab s+1 and this step.
    auto do_step = [&](auto rc, auto first_c, auto slots_c, bool last_iter, bool stores) SPECV_INLINE {
        constexpr int r = decltype(rc)::value;        // ring slot of slab s
        constexpr int rp = (r + 3) % RW;              // ring slot of slab s-1 = of slab s+3
        constexpr bool FIRST = decltype(first_c)::value;
        constexpr int SLOTS = decltype(slots_c)::value;
        if constexpr (ROWS) weave_rows(rc, slots_c);
        constexpr int g0 = r * 2 * TM;                // running group index (8 TM groups of 4 steps are a multiple of kHfRing)
        static_for<2 * TM>([&](auto ic) SPECV_INLINE {
            constexpr int i = decltype(ic)::value, t = i / TM, tm = i % TM;
            const bf16x8 h = hfq[(g0 + i) % kHfRing];
            if (tm < TM - 1 || full_tm) {             // wave-uniform
#pragma unroll
                for (int tn = 0; tn < SLOTS; ++tn) {
                    if constexpr (FIRST && t == 0 && tm >= 16)
                        asm("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc[tn][tm]) : "v"(wreg[r][t][tn]), "v"(h));
                    else if constexpr (tm >= 16)
                        asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[tn][tm]) : "v"(wreg[r][t][tn]), "v"(h));
                    else if constexpr (FIRST && t == 0)
                        asm("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[tn][tm]) : "v"(wreg[r][t][tn]), "v"(h));
                    else
                        asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[tn][tm]) : "v"(wreg[r][t][tn]), "v"(h));
                }
            }
            if constexpr (i < kHfCatchUp) {
                hfq[(g0 + kHfCross + 2 * i) % kHfRing] = hfrag(rc, std::integral_constant<int, kHfCross + 2 * i>{});
                hfq[(g0 + kHfCross + 2 * i + 1) % kHfRing] = hfrag(rc, std::integral_constant<int, kHfCross + 2 * i + 1>{});
            } else if constexpr (i + kHfAhead < 2 * TM) {
                hfq[(g0 + i + kHfAhead) % kHfRing] = hfrag(rc, std::integral_constant<int, i + kHfAhead>{});
            } else if constexpr (i >= 2 * TM - kHfCross) {
                hfq[(g0 + i + kHfCross) % kHfRing] =
                    hfrag(std::integral_constant<int, (r + 1) % RW>{}, std::integral_constant<int, i + kHfCross - 2 * TM>{});
            }
            if constexpr (i < SLOTS) fetch_w1(rp, 1, i);
            else if constexpr (i >= 4 && i < 4 + QN) stage_h1(rp, i - 4);
            else if constexpr (i >= TM && i < TM + SLOTS) fetch_w1(r, 0, i - TM);
            if constexpr (i == 4) {                   // W goes on to slab s+4: after the last one of a pass, to the next pass's panels
                wpos += kWSlab;
                if (r == 0 && last_iter) open_panels(p0_next, np_next);
            }
            if constexpr (i == TM - 1) {              // hidden goes on to slab s+4; after the last one, to slab 0 again
                hsrc += kMfSlab * 2;
                if (r == 0 && last_iter) hsrc = A;
            }
            if constexpr (i == 2 * TM - kHfCross - 1) {
                // Slab s+1 must be complete in LDS before anybody reads it.  This wave's share was requested in groups 4.. of
                // step s-2; younger than it are SLOTS W loads of that step and the 2 SLOTS + QN requests of each of the two steps since
                // (more where those steps were of a pass with more slots).
                // Where a tile was stored by counted stores in between, 4 for each of its TM or TM - 1 row tiles are younger still, and
                // waiting for all but 63 (the most the counter holds) lets them drain for two steps.  No LDS read of slab s is pending either: its slot may be overwritten.
                constexpr int kYounger = 2 * QN + 5 * SLOTS;
                constexpr int kDrain = kYounger + 4 * (TM - 1) < 63 ? kYounger + 4 * (TM - 1) : 63;
                static_assert(kYounger < 63, "s_waitcnt vmcnt has 6 bits");
                if (stores) __builtin_amdgcn_s_waitcnt(0x0070 | (kDrain & 15) | ((kDrain >> 4) << 14));
                else __builtin_amdgcn_s_waitcnt(0x0070 | (kYounger & 15) | ((kYounger >> 4) << 14));
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto do_steps = [&](auto first_c, auto slots_c, bool last_iter, bool stores) SPECV_INLINE {
        constexpr bool FIRST = decltype(first_c)::value;
        do_step(std::integral_constant<int, 0>{}, first_c, slots_c, last_iter, FIRST && stores);
        do_step(std::integral_constant<int, 1>{}, std::false_type{}, slots_c, false, FIRST && stores);
        do_step(std::integral_constant<int, 2>{}, std::false_type{}, slots_c, false, false);
        do_step(std::integral_constant<int, 3>{}, std::false_type{}, slots_c, false, false);
    };
    // Stores the finished tile of pass `pass`; returns whether it did so by exactly 4 stores per row tile.
    auto store_tile = [&](int pass, int st_p0, int st_np, auto slots_c) SPECV_INLINE {
        constexpr int SLOTS = decltype(slots_c)::value;
        const bool whole = !SUMMARY && st_np > 0 && (st_p0 + st_np) * 16 <= V;
        // acc[tn][tm][i] = C[row 16 tm + l16][entry 16 (st_p0 + tn) + 4 kg + i]
        // (SUMMARY) block of this wave and pass; its span is written once, by the first row group
        int blk = 0, count = 0;
        if constexpr (SUMMARY) {
            blk = (range * sm.passes_per_range + pass) * kMfWaves + wave;
            const int first = st_p0 * 16;
            count = max(0, min(st_np * 16, V - first));
            if (group == 0 && lane == 0) { sm.blk_span[2 * blk] = first; sm.blk_span[2 * blk + 1] = count; }
        }
        // (the lane's coordinates are taken afresh here: as invariants of the pass loop they, and everything derived from them, would
        // be kept in registers that the main loop needs)
        int lane_e = lane;
        asm volatile("" : "+v"(lane_e));
        const int l16_e = lane_e & 15, kg_e = lane_e >> 4;
        if (whole) {
            // All entries of the wave's panels are in the matrix: stores without tests, the next row tile written to the patch before
            // this one's stores wait for their reads.  Lanes past the wave's panels or the group's rows repeat the last entries or row.
            const int srow = lane_e >> 4, scol = min((lane_e & 15) * 4, st_np * 16 - 4);
            unsigned char* dst = reinterpret_cast<unsigned char*>(C + st_p0 * 16);
            const uint32_t off = ((uint32_t)srow * (uint32_t)V + (uint32_t)scol) * 4u;
            const size_t row_step = 16 * (size_t)V;
            f32x4 v[4];
            auto put = [&](auto tmc) SPECV_INLINE {
#pragma unroll
                for (int tn = 0; tn < SLOTS; ++tn)
                    *reinterpret_cast<f32x4*>(patch + patch_at(l16_e, tn * 4 + kg_e)) = acc[tn][decltype(tmc)::value];
            };
            put(std::integral_constant<int, 0>{});
            static_for<TM>([&](auto tmc) SPECV_INLINE {
                constexpr int tm = decltype(tmc)::value;
                if (tm < TM - 1 || full_tm) {         // wave-uniform
                    constexpr bool RAGGED = tm >= TM - 2;      // the group's last tile
                    const int last = M - 1 - tm * 16;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int prow = RAGGED ? min(q * 4 + srow, last) : q * 4 + srow;
                        v[q] = *reinterpret_cast<const f32x4*>(patch + patch_at(prow, scol >> 2));
                    }
                    if constexpr (tm + 1 < TM) { if (tm + 1 < TM - 1 || full_tm) put(std::integral_constant<int, tm + 1>{}); }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        f32x4_any* d = reinterpret_cast<f32x4_any*>(dst + off);
                        if constexpr (RAGGED) d = reinterpret_cast<f32x4_any*>(C + (size_t)(tm * 16 + min(q * 4 + srow, last)) * V + (st_p0 * 16 + scol));
                        if constexpr (NT) __builtin_nontemporal_store((f32x4_any)v[q], d); else *d = v[q];
                        dst += row_step;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        } else {                                      // (the summary instantiations are only launched for V % 4 == 0)
            // The tile is turned through the wave's own LDS patch so that one store instruction writes all
            // the wave's entries of a row (256 bytes), 4 rows at a time.  LDS operations of one wave execute in order, so
            // the patch needs no barrier and no second copy.
            constexpr int kLanesPerRow = kMfTN * 4, kRowsPerStore = 64 / kLanesPerRow;
            const int srow = lane_e / kLanesPerRow, scol = (lane_e % kLanesPerRow) * 4;     // this lane's row and entry when storing
            const int col0 = st_p0 * 16 + scol;
            const bool col_ok = scol < st_np * 16 && col0 + 4 <= V;
            const int col_tail = scol < st_np * 16 && !col_ok ? V - col0 : 0;
            uint32_t off = ((uint32_t)srow * (uint32_t)V + (uint32_t)col0) * 4u;
            int row = srow;                           // (running, for the same reason)
            const uint32_t row_step = (uint32_t)kRowsPerStore * 4u * (uint32_t)V;
            // (SUMMARY) running element index of this lane's row in blk_max / blk_sum, stepped like `off`: computed afresh
            // per row it is invariant from pass to pass, and the compiler would keep all 4 TM of them in registers
            uint32_t sat = (uint32_t)(row0 + srow) * (uint32_t)sm.blocks + (uint32_t)blk;
            const uint32_t sat_step = (uint32_t)kRowsPerStore * (uint32_t)sm.blocks;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                f32x4 t[SLOTS];
#pragma unroll
                for (int tn = 0; tn < SLOTS; ++tn) {
                    t[tn] = acc[tn][tm];
                    *reinterpret_cast<f32x4*>(patch + patch_at(l16_e, tn * 4 + kg_e)) = t[tn];
                }
#pragma unroll
                for (int q = 0; q < 16 / kRowsPerStore; ++q) {
                    const int prow = q * kRowsPerStore + srow;
                    const f32x4 v = *reinterpret_cast<const f32x4*>(patch + patch_at(prow, scol >> 2));
                    if constexpr (SUMMARY) {
                        // In this layout a row's 64 entries lie in the 16 lanes of one 16-lane row, 4 consecutive entries
                        // each (the values are in registers for the store anyway; taking them from the accumulators instead
                        // needs 16 more registers per tile, which this kernel does not have).  Entries past the block do not
                        // count.  Rotations within the 16-lane row leave the full maximum / sums in every lane.
                        // scale = log2(e)/T of a sampled row; a greedy row gets 1 so that its sum, which nobody reads as a
                        // sum, still turns NaN when the block holds a NaN (fmaxf drops NaNs, the exponential does not)
                        const float rs = row_scale[row];
                        const float scale = rs > 0.0f ? rs : 1.0f;
                        const int lim = count - scol;
                        float x[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = e < lim ? v[e] : -INFINITY;
                        const float m = row16_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
                        const float base = m > -INFINITY ? m : 0.0f;
                        float z = 0.0f;
#pragma unroll
                        for (int e = 0; e < 4; ++e) z += __builtin_amdgcn_exp2f((x[e] - base) * scale);
                        z = row16_sum(z);
                        if ((lane & 15) == 0 && row < M) {
                            sm.blk_max[sat] = z != z ? z : m;
                            sm.blk_sum[sat] = rs > 0.0f ? z : 0.0f;
                        }
                        sat += sat_step;
                        asm volatile("" : "+v"(sat));
                    }
                    if (row < M && col_ok) {
                        f32x4_any* dst = reinterpret_cast<f32x4_any*>(reinterpret_cast<unsigned char*>(C) + off);
                        if constexpr (NT) __builtin_nontemporal_store((f32x4_any)v, dst); else *dst = v;
                    }
                    if (!SUMMARY && row < M && col_tail > 0) {          // the matrix ends inside these four entries
                        float* dst = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(C) + off);
#pragma unroll
                        for (int e = 0; e < 3; ++e) if (e < col_tail) dst[e] = v[e];
                    }
                    off += row_step;                  // one running byte offset (rows x V x 4 < 2^32 per group)
                    row += kRowsPerStore;
                    asm volatile("" : "+v"(off), "+v"(row));
                }
                // one row tile at a time: left to itself the scheduler interleaves the summaries of all tiles, and their
                // temporaries (16 values each) no longer fit beside the W ring
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        return whole;
    };

    // The last pass of a range, which has 1..16 panels, is in code of its own for two and for three panels per wave: no branches, and waits that count
    // its requests (a wave that owns fewer repeats its last panel).  One code for any number, with a run-time test of the wave's panels in every
    // group -> these, us: V = 151936, H = 4096 M = 188 262 -> 247, M = 576 619 -> 606, M = 1152 1161 -> 1148; V = 32000 M = 188 76 -> 59.  Where ways with
    // and without the fourth panel meet, the compiler would also move the whole ring to other registers, and wait for every request in flight to do so.
    // In each, the first four steps stand outside the loop: there, and only there, the waits know of the stores of the tile before.
    bool stored = false;                              // a tile's counted stores precede this pass
    auto one_pass = [&](auto slots_c) SPECV_INLINE {
        do_steps(std::true_type{}, slots_c, nslab == RW, stored);
        for (int s = RW; s < nslab; s += RW) do_steps(std::false_type{}, slots_c, s + RW == nslab, false);
        // the tile is complete; the next pass's first slabs are already in flight
        stored = store_tile(pass, wave_p0, wave_np, slots_c);
    };
    // (beyond 16 row tiles the code for three leaves the compiler short of registers: it moves accumulators inside the steps; four serve it)
    constexpr bool THREE = TM <= 16;
    const int slots = !THREE && mf_last_slots(n_own) == 3 ? kMfTN : mf_last_slots(n_own);
    const int full = mf_full_passes(p_begin, p_end, V), four = slots == kMfTN ? npass : full;      // (full: npass or npass - 1)
    while (pass < four) {
        one_pass(std::integral_constant<int, kMfTN>{});
        ++pass;
        wave_p0 = p0_next; wave_np = np_next;
        pass_panels(min(pass + 1, npass - 1), p0_next, np_next);
    }
    if (slots == 2) one_pass(std::integral_constant<int, 2>{});
    if constexpr (THREE) { if (slots == 3) one_pass(std::integral_constant<int, 3>{}); }
    if constexpr (SUMMARY) {                          // block slots of passes this range does not have
        if (group == 0)
            for (int b = npass * kMfWaves + tid; b < sm.passes_per_range * kMfWaves; b += 64 * kMfWaves) {
                sm.blk_span[2 * (range * sm.passes_per_range * kMfWaves + b)] = 0;
                sm.blk_span[2 * (range * sm.passes_per_range * kMfWaves + b) + 1] = 0;
            }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);               // no direct load of this wave is still landing when the LDS is given up
}

// 9 to 16 row tiles per group
template <int TM, MfmaLoads LOADS, bool NT, bool SUMMARY>
__global__ __launch_bounds__(64 * kMfWaves, 1) void lm_head_mfma_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ Wp, float* __restrict__ C, int M, int H, int V, int n_panels, int panels_per_wg,
    int groups, int tiles_lo, int groups_hi, LmSummary sm)
{
    lm_head_mfma_tiles<TM, LOADS, NT, SUMMARY>(A, Wp, C, M, H, V, n_panels, panels_per_wg, groups, tiles_lo, groups_hi, sm);
}

// 8 (and 9 and 10 with nontemporal loads): one group of 113 to 160 rows; 17 and 18: 16 tiles of accumulators fill the accumulation registers, the others are
// vector registers, and LDS is full to the byte
template <int TM, MfmaLoads LOADS, bool NT>
__global__ __launch_bounds__(64 * kMfWaves, 1) void lm_head_tile_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ Wp, float* __restrict__ C, int M, int H, int V, int n_panels, int panels_per_wg,
    int groups, int tiles_lo, int groups_hi)
{
    lm_head_mfma_tiles<TM, LOADS, NT, false>(A, Wp, C, M, H, V, n_panels, panels_per_wg, groups, tiles_lo, groups_hi, LmSummary{});
}

// 8 to 16, W row-major
template <int TM, MfmaLoads LOADS, bool NT>
__global__ __launch_bounds__(64 * kMfWaves, 1) void lm_head_rowmajor_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ W, float* __restrict__ C, int M, int H, int V, int n_panels, int panels_per_wg,
    int groups, int tiles_lo, int groups_hi)
{
    lm_head_mfma_tiles<TM, LOADS, NT, false>(A, W, C, M, H, V, n_panels, panels_per_wg, groups, tiles_lo, groups_hi, LmSummary{});
}

template <int TM, MfmaLoads LOADS, bool NT, bool SUMMARY>
static int launch_mfma(const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, LmSummary sm, hipStream_t s)
{
    constexpr size_t smem = mf_lds_bytes(TM, SUMMARY);
    static LdsGrantTable granted = {};
    if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(&lm_head_mfma_kernel<TM, LOADS, NT, SUMMARY>), smem, granted, "spec_lm_head_packed")) return rc;
    hipLaunchKernelGGL((lm_head_mfma_kernel<TM, LOADS, NT, SUMMARY>), dim3(L.ranges * L.groups), dim3(64 * kMfWaves), smem, s, a, wp, c, M, H, V,
                       (V + 15) / 16, L.per_range, L.groups, L.tiles_lo, L.groups_hi, sm);
    return SPEC_OK;
}

// The instantiations for TM..16 row tiles of one kind of loads: a file each, built side by side.
template <MfmaLoads LOADS, bool SUMMARY, int TM>
static int launch_mfma_tiles(bool nt, const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, const LmSummary& sm, hipStream_t s)
{
    if (L.tm == TM)
        return nt ? launch_mfma<TM, LOADS, true, SUMMARY>(a, wp, c, M, H, V, L, sm, s) : launch_mfma<TM, LOADS, false, SUMMARY>(a, wp, c, M, H, V, L, sm, s);
    if constexpr (TM < 16) return launch_mfma_tiles<LOADS, SUMMARY, TM + 1>(nt, a, wp, c, M, H, V, L, sm, s);
    else return fail(SPEC_ESHAPE, "spec_lm_head_packed: no large-tile instantiation for %d row tiles per group", L.tm);
}

template <int TM, MfmaLoads LOADS, bool NT>
static int launch_tile(const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s)
{
    constexpr size_t smem = mf_lds_bytes(TM, false);
    static_assert(smem <= 160 * 1024, "the LDS of a CU");
    static LdsGrantTable granted = {};
    if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(&lm_head_tile_kernel<TM, LOADS, NT>), smem, granted, "spec_lm_head_packed")) return rc;
    hipLaunchKernelGGL((lm_head_tile_kernel<TM, LOADS, NT>), dim3(L.ranges * L.groups), dim3(64 * kMfWaves), smem, s, a, wp, c, M, H, V,
                       (V + 15) / 16, L.per_range, L.groups, L.tiles_lo, L.groups_hi);
    return SPEC_OK;
}

template <int TM, MfmaLoads LOADS, bool NT>
static int launch_rowmajor(const uint16_t* a, const uint16_t* w, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s)
{
    if (L.tm == TM) {
        constexpr size_t smem = mf_lds_bytes(TM, false);
        static LdsGrantTable granted = {};
        if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(&lm_head_rowmajor_kernel<TM, LOADS, NT>), smem, granted, "spec_lm_head")) return rc;
        hipLaunchKernelGGL((lm_head_rowmajor_kernel<TM, LOADS, NT>), dim3(L.ranges * L.groups), dim3(64 * kMfWaves), smem, s, a, w, c, M, H, V,
                           (V + 15) / 16, L.per_range, L.groups, L.tiles_lo, L.groups_hi);
        return SPEC_OK;
    }
    if constexpr (TM < 16) return launch_rowmajor<TM + 1, LOADS, NT>(a, w, c, M, H, V, L, s);
    else return fail(SPEC_ESHAPE, "spec_lm_head: no large-tile instantiation for %d row tiles per group", L.tm);
}

int lm_head_tile(MfmaLoads loads, bool nt, const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, hipStream_t s);

#define SPECV_MFMA_FILE(name) int name(bool nt, const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const MfmaLayout& L, const LmSummary& sm, hipStream_t s)
SPECV_MFMA_FILE(lm_head_mfma_buffer);
SPECV_MFMA_FILE(lm_head_mfma_global);
SPECV_MFMA_FILE(lm_head_mfma_stream);      // 11 row tiles or more (one group of more than 160 rows)
SPECV_MFMA_FILE(lm_head_mfma_summary);     // (buffer loads)

}  // namespace specv
