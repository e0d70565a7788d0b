// spec_lm_head_pack / spec_lm_head_packed: the logits of every candidate row (paper, Appendix "Target side":
// every position of the verification candidate is scored) with the vocabulary matrix stored once, at load
// time, in the order the matrix cores consume it.
//
// Why a second layout.  With W row-major the weight stream of a verify batch touches, per workgroup pass, one
// 64-byte piece of each of 128 rows that lie 2*H bytes apart; measured on MI355X that stream reaches 4.4-4.9
// TB/s, falls further when more rows are open, and the L2-resident hidden rows that every pass re-reads cost
// their transfer time on top.  Stored as below, every wave load is 1 KB of consecutive bytes, the stream runs at
// the rate of a linear read (6.0 TB/s), and because the number of open rows no longer matters a pass can be
// twice as wide, which halves the hidden re-reads.
//
// Packed layout: panels of 16 vocabulary entries; panel p, k-tile t (32 consecutive k), lane l, element j:
//     Wp[((p * (H/32) + t) * 64 + l) * 8 + j] = W[16 p + l % 16][32 t + 8 (l / 16) + j]      (0 for entries >= V)
// i.e. the A operand of v_mfma_f32_16x16x32_bf16 for that tile, lane by lane.  ceil(V/16) panels.
#include "common.h"
#include "lm_head_tiles.h"

#include <type_traits>

namespace specv {

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // (a row of logits starts at any multiple of 4 bytes)

constexpr int kPkSlab = 128;                   // k per hidden slab in LDS
constexpr int kPkHPitch = kPkSlab * 2;         // bytes per hidden row in LDS; 16-byte chunk ch of row r sits at position ch ^ (r & 15)
constexpr int kPkMaxRows = 160;                // rows of hidden per row group (one workgroup's share)

__global__ __launch_bounds__(256) void lm_head_pack_kernel(const uint16_t* __restrict__ W, uint16_t* __restrict__ Wp,
                                                           int V, int H, size_t n_chunks)
{
    // one 16-byte chunk of the packed matrix per thread and step: consecutive threads write consecutive chunks
    const int ktiles = H / 32;
    for (size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x; o < n_chunks; o += (size_t)gridDim.x * blockDim.x) {
        const int lane = (int)(o & 63);
        const size_t tile = o >> 6;
        const int t = (int)(tile % ktiles);
        const size_t p = tile / ktiles;
        const size_t entry = p * 16 + (lane & 15);
        u32x4 v = {0u, 0u, 0u, 0u};
        if (entry < (size_t)V) v = *reinterpret_cast<const u32x4*>(W + entry * H + t * 32 + (lane >> 4) * 8);
        *reinterpret_cast<u32x4*>(Wp + o * 8) = v;
    }
}

// ------------------------------------------------------------------------------------------------
// One persistent workgroup of NW waves per CU owns a contiguous range of panels and walks it in passes of at most
// NW * TN panels (16 = 256 vocabulary entries by default), cut so that all passes of a workgroup are equally wide
// (whatever V is, every CU streams at the same rate to the end).  Inside a pass wave w takes up to TN consecutive
// panels and all rows of hidden; with NW = 8 two waves share each SIMD and one's MFMAs cover the other's waits
// (10 us of 297 at M = 160):
//   * W goes from HBM straight into registers in operand order through a ring of RS slabs of 128 k, refilled
//     right after the MFMAs that consumed a chunk pair; no W byte touches LDS.
//   * hidden is staged through LDS in 128-k slabs shared by the waves, requested two slabs ahead: loads retire
//     in order, so a younger hidden load must never be what the math waits for.
//   * the next pass's first loads are issued before the finished tile is stored, because stores share the
//     in-order queue with loads.
//   * C^T tiles come out with 4 consecutive vocabulary entries per lane and 16 rows per instruction; they are
//     turned through LDS so that a store instruction writes whole 128-byte lines (all the wave's entries of a
//     row, 128 or 256 bytes).  With one or two row groups they are stored nontemporal (nobody reads them before the
//     next kernel; 263 against 280 us at M = 160); with many groups the L2 absorbs the writes better (1351 against
//     1504 us at M = 1152).
// TM: 16-row tiles of hidden per row group (rows <= 16 TM); RS: slabs in the W register ring (1, or 2 with 4 waves of 2 panels: with 8 waves 2
// measured 5 us slower at M = 160 and equal above); NW: waves (4 or 8); NT: nontemporal stores of the logits;
// TN: panels per wave and pass (2 or 4: a pass is 16 NW TN entries wide);
// ROWS: W row-major instead of packed: a load takes 128 bytes of 8 rows (whole lines) and weave_rows makes operands of two of them;
// SW: W by nontemporal loads (one row group and a matrix too large for the memory-side cache);
// STATS: also leave per-block maxima for greedy acceptance.
// ------------------------------------------------------------------------------------------------
template <int TM, int RS, int NW, bool NT, int TN, bool STATS, bool SW, bool RAGGED, bool ROWS>
__global__ __launch_bounds__(64 * NW, 1) void lm_head_packed_kernel(
    const uint16_t* __restrict__ A_all, const uint16_t* __restrict__ Wp, float* __restrict__ C_all,
    int M_all, int H, int V, int n_panels, int panels_per_wg, int groups, int rows_per_group,
    float* __restrict__ blk_max, int32_t* __restrict__ blk_arg, int nblk, int passes_per_range)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int kPassPanels = NW * TN;              // panels per workgroup pass
    constexpr int kThreads = 64 * NW;
    constexpr int BM = TM * 16;                       // hidden rows staged in LDS (rows >= M repeat row M-1)
    constexpr int H_LOADS = (BM * 16 + kThreads - 1) / kThreads;   // 16-byte chunks of a hidden slab per thread
    constexpr int kRing = 4 * RS;
    constexpr int kHfAhead = 4;                       // (8 is slower: 340 against 325 us at M = 160)
    constexpr int U = RS % 2 ? 2 * RS : RS;           // slabs per unrolled step: even, so that buffer parities are static
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, l16 = lane & 15, kg = lane >> 4;
    // Workgroup -> (row group, panel range).  Workgroups are dealt round-robin to the 8 XCDs, each with its own L2:
    // the row groups of one panel range sit on the same XCD and are dispatched together, so that they stream the
    // same panels at the same time and all but the first read of a panel is an L2 hit.
    const int xcd = blockIdx.x & 7, dealt = blockIdx.x >> 3;
    const int group = dealt % groups, range = (dealt / groups) * 8 + xcd;
    const int M = min(rows_per_group, M_all - group * rows_per_group);              // >= 1 by the host's choice of groups
    const uint16_t* __restrict__ A = A_all + (size_t)group * rows_per_group * H;
    float* __restrict__ C = C_all + (size_t)group * rows_per_group * V;
    const int p_begin = range * panels_per_wg;
    const int p_end = min(n_panels, p_begin + panels_per_wg);
    // STATS: block b = range * passes_per_range + pass of a row holds the maximum of the logits this workgroup computed
    // for the row in that pass and its lowest index (NaN / INT_MAX if the block holds a NaN, -inf / INT_MAX for a
    // block without entries), so that greedy acceptance need not read the logits again.
    auto fill_empty_blocks = [&](int first_pass) {
        const int missing = passes_per_range - first_pass;
        for (int e = tid; e < missing * M; e += kThreads) {
            const int r = e / missing, q = e - r * missing;
            const size_t o = (size_t)(group * rows_per_group + r) * nblk + (size_t)range * passes_per_range + first_pass + q;
            blk_max[o] = -INFINITY;
            blk_arg[o] = 0x7FFFFFFF;
        }
    };
    if (p_begin >= p_end) {
        if (STATS) fill_empty_blocks(0);
        return;
    }
    const int n_own = p_end - p_begin;
    const int npass = (n_own + kPassPanels - 1) / kPassPanels;

    f32x4 acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = f32x4{0.f, 0.f, 0.f, 0.f};

    const uint16_t* wptr[TN];
    const uint16_t* wptr_hi[ROWS ? TN : 1];
    u32x4 wreg[TN][kRing], hreg[2][H_LOADS];
    int wave_p0 = 0, wave_np = 0;
    auto open_pass = [&](int pass) {                  // the wave's panels of a pass and their stream pointers
        const int lo = p_begin + (int)((long)pass * n_own / npass);
        const int hi = p_begin + (int)((long)(pass + 1) * n_own / npass);      // 1 <= hi - lo <= kPassPanels
        const int m = hi - lo;
        wave_p0 = lo + wave * m / NW;
        wave_np = lo + (wave + 1) * m / NW - wave_p0; // 0 .. TN; wave_p0 < hi is a panel of the matrix either way
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            // panels past the wave's share re-read its last one (branch-free loop); their results are never stored
            const int p = wave_p0 + max(0, min(tn, wave_np - 1));
            if constexpr (ROWS) {
                // entries past V repeat the last one; which half of a row's 128 bytes the lane takes: see weave_rows
                wptr[tn] = Wp + (size_t)min(p * 16 + (l16 & 7), V - 1) * H + (kg + (l16 & 8) / 2) * 8;
                wptr_hi[tn] = Wp + (size_t)min(p * 16 + 8 + (l16 & 7), V - 1) * H + (kg + 4 - (l16 & 8) / 2) * 8;
            } else {
                wptr[tn] = Wp + (size_t)p * 16 * H + lane * 8;
            }
        }
    };
    auto fetch_w = [&](int c, int slab) {             // chunk c of the ring <- k-tile 4 * slab + c % 4
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const uint16_t* at;
            if constexpr (ROWS) at = ((c & 1) ? wptr_hi[tn] : wptr[tn]) + (size_t)(slab * 2 + ((c & 3) >> 1)) * 64;
            else at = wptr[tn] + (size_t)(slab * 4 + (c & 3)) * 512;
            const u32x4* src = reinterpret_cast<const u32x4*>(at);
            if constexpr (SW) wreg[tn][c] = __builtin_nontemporal_load(src); else wreg[tn][c] = *src;
        }
    };
    // (ROWS) Chunks c, c + 1 of the ring as loaded hold 128 bytes of rows 0..7 and of rows 8..15 of a panel: lane (l16, kg) of the first
    // has row l16 % 8, 16-byte piece kg (l16 < 8) or 4 + kg (else); of the second row 8 + l16 % 8, piece 4 + kg or kg.  Here they become the
    // operands of the k-tiles they cover: row l16, piece kg (a selection), and row l16, piece 4 + kg (selection, then a rotation by 8
    // within the 16 lanes).
    auto weave_rows = [&](int c) {
        const bool low = l16 < 8;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t a = wreg[tn][c][e], b = wreg[tn][c + 1][e];
                wreg[tn][c][e] = low ? a : b;
                wreg[tn][c + 1][e] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(low ? b : a), 0x128, 0xF, 0xF, false);   // row_ror:8
            }
    };
    auto fetch_h = [&](int set, int k0) {
#pragma unroll
        for (int p = 0; p < H_LOADS; ++p) {
            // rows past M read row M-1: every output row depends on its own hidden row only
            const int idx = min(tid + p * kThreads, BM * 16 - 1), row = min(idx >> 4, M - 1), ch = idx & 15;
            hreg[set][p] = *reinterpret_cast<const u32x4*>(A + (size_t)row * H + k0 + ch * 8);
        }
    };
    auto stash_h = [&](int set, unsigned char* buf) {
#pragma unroll
        for (int p = 0; p < H_LOADS; ++p) {
            const int idx = min(tid + p * kThreads, BM * 16 - 1), row = idx >> 4, ch = idx & 15;
            *reinterpret_cast<u32x4*>(buf + row * kPkHPitch + ((ch ^ (row & 15)) << 4)) = hreg[set][p];
        }
    };
    const int nslab = H / kPkSlab;                    // multiple of U
    // first requests of a pass, in the order of the steady state (hidden slab, then W chunks)
    auto open_loads = [&]() {
        fetch_h(0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) fetch_w(c, 0);
        fetch_h(1, kPkSlab);                          // slab 1, stashed at the end of slab 0
#pragma unroll
        for (int c = 4; c < kRing; ++c) fetch_w(c, c >> 2);
    };

    unsigned char* buf0 = smem;
    unsigned char* buf1 = smem + BM * kPkHPitch;
    constexpr int kPatchPitch = TN * 64 + 16;         // bytes per row of the wave's store patch: 16 rows x 16 TN entries
    unsigned char* patch = smem + 2 * BM * kPkHPitch + wave * (16 * kPatchPitch);
    // STATS: per row one candidate (value, index) from each wave, merged by the first threads after the next barrier
    float* cand_v = reinterpret_cast<float*>(smem + 2 * BM * kPkHPitch + NW * 16 * kPatchPitch);   // [BM][NW]
    int* cand_i = reinterpret_cast<int*>(cand_v + BM * NW);
    auto merge_candidates = [&](int done_pass) {          // after a barrier that follows the pass's candidate writes
        for (int r = tid; r < M; r += kThreads) {
            float best = -INFINITY;
            int bi = 0x7FFFFFFF;
            bool nan = false;
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                const float v = cand_v[r * NW + q];
                const int vi = cand_i[r * NW + q];
                nan |= (v != v);
                if (v > best || (v == best && vi < bi)) { best = v; bi = vi; }
            }
            const size_t o = (size_t)(group * rows_per_group + r) * nblk + (size_t)range * passes_per_range + done_pass;
            blk_max[o] = nan ? __builtin_nanf("") : best;
            blk_arg[o] = nan ? 0x7FFFFFFF : bi;
        }
    };
    int pass = 0;
    open_pass(pass);
    open_loads();
    for (;;) {
        stash_h(0, buf0);                             // every wave left the previous pass through a barrier
        __syncthreads();
        if (STATS && pass > 0) merge_candidates(pass - 1);   // written before this barrier, rewritten 2 * nslab barriers later
        for (int sR = 0; sR < nslab; sR += U) {
#pragma unroll
            for (int par2 = 0; par2 < U; ++par2) {
                const int s = sR + par2, par = par2 % RS;
                unsigned char* cur = (s & 1) ? buf1 : buf0;
                unsigned char* nxt = (s & 1) ? buf0 : buf1;   // last read in slab s-1, before the barrier that ended it
                // past the end the prefetches wrap to a valid slab (cache hits, results unused): no branch in the loop
                const int kh = min((s + 2) * kPkSlab, H - kPkSlab);
                const int sw = min(s + RS, nslab - 1);
                fetch_h(s & 1, kh);
                // the scheduler must not move the loads: their program order is what the in-order wait counters
                // are derived from, so every step is fenced
                __builtin_amdgcn_sched_barrier(0);
                // The slab is 4 chunks x TM row tiles; each (chunk, row tile) fragment of hidden feeds the TN MFMAs of
                // the wave's panels and is read from LDS kHfAhead fragments before it is used: a short ring instead of
                // a whole chunk of fragments, which leaves the registers to the W ring.
                bf16x8 hfq[kHfAhead];
                auto hfrag = [&](int i) {
                    return *reinterpret_cast<const bf16x8*>(cur + ((i % TM) * 16 + l16) * kPkHPitch + ((((i / TM) * 4 + kg) ^ l16) << 4));
                };
#pragma unroll
                for (int i = 0; i < kHfAhead; ++i) hfq[i] = hfrag(i);
#pragma unroll
                for (int i = 0; i < 4 * TM; ++i) {
                    const int c = i / TM, tm = i % TM;
                    if (ROWS && tm == 0 && (c & 1) == 0) weave_rows(par * 4 + c);
                    const bf16x8 h = hfq[i % kHfAhead];
                    if (i + kHfAhead < 4 * TM) hfq[i % kHfAhead] = hfrag(i + kHfAhead);
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
                        // wave-uniform: a panel slot the wave does not own costs no MFMA.  The chip is power-limited under
                        // random bf16 operands, so the skipped work raises the clock for everything else (M = 160: 279
                        // against 295 us); with one wave per SIMD the branches cost more than they save (339 us).
                        if (NW == 4 || tn == 0 || tn < wave_np)
                            acc[tn][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wreg[tn][par * 4 + c]), h,
                                                                              acc[tn][tm], 0, 0, 0);
                    if (tm == TM - 1) {
                        if (c & 1) {                  // the chunk pair just consumed is requested again, RS slabs further
                            fetch_w(par * 4 + c - 1, sw);
                            fetch_w(par * 4 + c, sw);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                stash_h((s & 1) ^ 1, nxt);            // slab s+1, requested one slab ago
                __syncthreads();
            }
        }
        const int st_p0 = wave_p0, st_np = wave_np;
        ++pass;
        const bool more = pass < npass;
        if (more) {
            open_pass(pass);
            open_loads();
            __builtin_amdgcn_sched_barrier(0);
        }
        // acc[tn][tm][i] = C[row 16 tm + l16][entry 16 (st_p0 + tn) + 4 kg + i]
        if (STATS) {
            int cslot = l16 * NW + wave;                  // a running slot: ten addresses kept across the pass would spill
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                float best = -INFINITY;
                int bi = 0x7FFFFFFF;
                bool nan = false;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int e = (st_p0 + tn) * 16 + kg * 4 + i;
                        const float v = acc[tn][tm][i];
                        if (tn < st_np && e < V) {       // ascending e: the first maximum is the lowest index
                            nan |= (v != v);
                            if (v > best) { best = v; bi = e; }
                        }
                    }
#pragma unroll
                for (int sh = 16; sh <= 32; sh <<= 1) {   // the four lanes of a row
                    const float ov = __shfl_xor(best, sh, 64);
                    const int oi = __shfl_xor(bi, sh, 64);
                    nan |= (bool)__shfl_xor((int)nan, sh, 64);
                    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
                }
                if (kg == 0) {
                    cand_v[cslot] = nan ? __builtin_nanf("") : best;
                    cand_i[cslot] = bi;
                }
                cslot += 16 * NW;
                asm volatile("" : "+v"(cslot));
            }
        }
        {
            // The tile is turned through the wave's own LDS patch so that one store instruction writes
            // all the wave's entries of a row (whole cache lines where rows are aligned), 4 or 8 rows at a time, instead of 64 bytes of each of 16 rows.
            // LDS operations of one wave execute in order, so the patch needs no barrier and no second copy.  A row starts at any multiple of 4 bytes; the last
            // entries of one whose length is no multiple of 4 are stored one by one.  (All entries one by one there: V = 50021, H = 1280 M = 57 30.1 -> 27.0 us,
            // M = 96 35.8 -> 31.8; V = 32001, H = 1024 M = 60 20.4 -> 16.9.)  Whole rows (not RAGGED) have kernels of their own: through the code with tails V = 64000, H = 512 M = 144
            // 20.7 -> 21.6, V = 44000 15.1 -> 15.7; with both codes in one kernel V = 32000, H = 1024 M = 20 12.8 -> 13.2.
            constexpr int kLanesPerRow = TN * 4, kRowsPerStore = 64 / kLanesPerRow;
            const int srow = lane / kLanesPerRow, scol = (lane % kLanesPerRow) * 4;     // this lane's row and entry when storing
            const int col0 = st_p0 * 16 + scol;
            uint32_t off = ((uint32_t)srow * (uint32_t)V + (uint32_t)col0) * 4u;
            const uint32_t row_step = (uint32_t)kRowsPerStore * 4u * (uint32_t)V;
            const bool mine = scol < st_np * 16, col_ok = mine && (RAGGED ? col0 + 4 <= V : col0 < V);
            const int col_tail = RAGGED && mine && !col_ok ? V - col0 : 0;
            typedef typename std::conditional<RAGGED, f32x4_any, f32x4>::type Quad;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) {
                    *reinterpret_cast<f32x4*>(patch + l16 * kPatchPitch + (tn * 16 + kg * 4) * 4) = acc[tn][tm];
                    acc[tn][tm] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int q = 0; q < 16 / kRowsPerStore; ++q) {
                    const int prow = q * kRowsPerStore + srow, row = tm * 16 + prow;
                    const f32x4 v = *reinterpret_cast<const f32x4*>(patch + prow * kPatchPitch + scol * 4);
                    if (row < M && col_ok) {
                        Quad* dst = reinterpret_cast<Quad*>(reinterpret_cast<unsigned char*>(C) + off);
                        if constexpr (NT) __builtin_nontemporal_store((Quad)v, dst); else *dst = v;
                    }
                    if (RAGGED && row < M && col_tail > 0) {      // the matrix ends inside these four entries
                        float* dst = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(C) + off);
#pragma unroll
                        for (int e = 0; e < 3; ++e) if (e < col_tail) dst[e] = v[e];
                    }
                    off += row_step;                  // one running byte offset (M * V * 4 < 2^32 per launch) instead of
                    asm volatile("" : "+v"(off));     // one row address per store kept alive across the whole pass
                }
            }
        }
        if (!more) break;
    }
    if (STATS) {
        __syncthreads();
        merge_candidates(npass - 1);
        fill_empty_blocks(npass);
    }
}

Tunable g_lm_packed_wide{0};      // benchmark hook: 512-entry passes for M <= 160 (0 = automatic, 1 = always, 2 = never)
Tunable g_lm_packed_waves{0};     // benchmark hook: waves per workgroup of the packed kernel (4 or 8; 0 = automatic)

// panel ranges and panels per range of a launch: ranges is a multiple of 8 (one per XCD and step of the dealing), as many
// as there are CUs per row group; trailing ranges without panels are dropped 8 at a time
static void packed_geometry(int V, int groups, int* ranges, int* per_range)
{
    const int cus = device_cu_count();
    const int n_panels = (V + 15) / 16;
    const int r0 = max(8, cus / groups / 8 * 8);
    *per_range = (n_panels + r0 - 1) / r0;
    *ranges = ((n_panels + *per_range - 1) / *per_range + 7) / 8 * 8;
}

template <int TM, int RS, int NW, bool NT, int TN, bool STATS, bool SW, bool RAGGED, bool ROWS>
static int launch_packed_as(const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, int groups, hipStream_t s,
                            float* blk_max, int32_t* blk_arg)
{
    constexpr int BM = TM * 16;
    const size_t smem = 2 * (size_t)BM * kPkHPitch + NW * 16 * (TN * 64 + 16) + (STATS ? (size_t)BM * NW * 8 : 0);
    static LdsGrantTable granted = {};
    if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(&lm_head_packed_kernel<TM, RS, NW, NT, TN, STATS, SW, RAGGED, ROWS>), smem, granted, ROWS ? "spec_lm_head" : "spec_lm_head_packed")) return rc;
    int ranges, per_range;
    packed_geometry(V, groups, &ranges, &per_range);
    const int ppr = (per_range + NW * TN - 1) / (NW * TN);
    hipLaunchKernelGGL((lm_head_packed_kernel<TM, RS, NW, NT, TN, STATS, SW, RAGGED, ROWS>), dim3(ranges * groups), dim3(64 * NW), smem, s, a, wp, c, M, H, V,
                       (V + 15) / 16, per_range, groups, BM, blk_max, blk_arg, ranges * ppr, ppr);
    return SPEC_OK;
}

static int panels_per_cu(int V)
{
    int ranges, per_range;
    packed_geometry(V, 1, &ranges, &per_range);
    return per_range;
}

// W is read once when one row group covers the batch.  A matrix above 3/8 of the memory-side cache is read nontemporal: it does not push the step's other
// operands out of that cache, and it would not be found there by the next step.  Measured on steps over three batches in turn, ordinary ->
// nontemporal, us: W = 97 MiB (V = 40001, H = 1280) 4 requests 50.3 -> 47.2, 32 requests 81.5 -> 75.9; 156 MiB (32000, 2560) 59.3 -> 54.4, 81.8 -> 77.1;
// 250 MiB (64000, 2048) 83.5 -> 78.7, 100.6 -> 96.9; 13 ragged requests on 122 MiB (50021, 1280) 92.5 -> 83.8; 1.16 GiB one request 267 -> 244; below
// the line, 73 MiB 48.0 -> 47.8.  (The LM head alone, called again and again on one matrix of 100 to 280 MiB, loses 3 to 15 % by it: 195 MiB, M = 40 34 -> 38.
// So does a batch of several row groups, which reads W from the L2 in all but one.)
// Row-major, alone on three matrices in turn: where rows are a multiple of 2 KB, or the waves have nearly all their panel slots to fill (H = 2560, M = 1:
// V = 64000, 16 panels of 16 59 -> 53, V = 128256, 2 x 16 113 -> 103; but V = 90000, 2 x 11 87 -> 93, V = 36000, 9 46 -> 51.5, V = 151936, 38 in 3
// passes 138 -> 143; H = 4096 V = 90000 156 -> 152, V = 151936 215 -> 203).
template <bool ROWS>
static bool stream_weights(int H, int V, int pass_panels)
{
    if ((size_t)V * H * 2 <= kMemorySideCache * 3 / 8) return false;
    if (!ROWS || H % 1024 == 0) return true;
    const int p = panels_per_cu(V), passes = (p + pass_panels - 1) / pass_panels;
    return p * 16 >= 13 * passes * pass_panels;
}

template <int TM, int RS, int NW, bool NT, int TN, bool STATS = false, bool ROWS = false>
static int launch_packed(const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, int groups, hipStream_t s,
                         float* blk_max = nullptr, int32_t* blk_arg = nullptr)
{
    if constexpr (NT) {
        if (groups == 1 && stream_weights<ROWS>(H, V, NW * TN))
            return V % 4 == 0 ? launch_packed_as<TM, RS, NW, NT, TN, STATS, true, false, ROWS>(a, wp, c, M, H, V, groups, s, blk_max, blk_arg)
                              : launch_packed_as<TM, RS, NW, NT, TN, STATS, true, true, ROWS>(a, wp, c, M, H, V, groups, s, blk_max, blk_arg);
    }
    return V % 4 == 0 ? launch_packed_as<TM, RS, NW, NT, TN, STATS, false, false, ROWS>(a, wp, c, M, H, V, groups, s, blk_max, blk_arg)
                      : launch_packed_as<TM, RS, NW, NT, TN, STATS, false, true, ROWS>(a, wp, c, M, H, V, groups, s, blk_max, blk_arg);
}

// A vocabulary of at most 8 panels per CU (V <= 32768 on 256 CUs) is one pass of 4 waves with 2 panels each and a 2-slab ring; 8 waves would have one
// panel each, their second slot re-reading it, and twice the LDS reads per panel.  Measured at V = 32000, 8 against 4 waves: H = 4096
// M = 40 51.6 -> 47.8 us, M = 160 70 -> 60; H = 2048 M = 96 35.3 -> 32.6; row-major H = 4096 M = 80 74 -> 48, M = 160 87 -> 61.
// With more panels 8 waves are ahead (V = 50021, H = 1280, M = 40: 27.5 against 30.5).
static bool few_panels(int V) { return panels_per_cu(V) <= 8; }

// The logits are stored nontemporal for one and two row groups, also where rows share lines with their neighbours (V no multiple of 16): followed by the acceptance that reads them,
// as in a step, ordinary -> nontemporal, us: V = 50021, H = 1280 M = 57 36.2 -> 35.6, M = 96 41.8 -> 41.8 (the LM head alone 26.2 -> 27.0, 30.3 -> 31.9); V = 100001, H = 4096 M = 57
// 160.7 -> 147.3, V = 151935 250 -> 228; row-major V = 64013, H = 4096 110.0 -> 110.6, V = 151935 272 -> 248.  But a vocabulary of at most 2 panels per CU, whose stores are all there is
// between the last product and the end: V = 2001, H = 1280 M = 16 6.0 -> 6.4, M = 57 8.6 -> 9.1, M = 96 11.7 -> 12.3; V = 8001 M = 16 6.5 -> 6.9, M = 57 9.6 -> 10.1.
static bool ordinary_stores(int H, int V) { return V % 16 != 0 && panels_per_cu(V) <= 2 && (size_t)V * H * 2 <= kMemorySideCache * 3 / 8; }

template <int TM>
static int launch_packed_auto(const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, int groups, hipStream_t s,
                              float* blk_max, int32_t* blk_arg)
{
    if (blk_max) {
        if (groups > 2) return launch_packed<TM, 1, 8, false, 2, true>(a, wp, c, M, H, V, groups, s, blk_max, blk_arg);
        return launch_packed<TM, 1, 8, true, 2, true>(a, wp, c, M, H, V, groups, s, blk_max, blk_arg);
    }
    // measured on MI355X at M = 160, V = 151936 inside the whole verify step: 8 waves 287 us, 4 waves 297 us (a 2-slab
    // W ring is 5 us slower with either); at M = 40 both take 218 us; at M = 576 and 1152 8 waves are 5 % ahead
    if (g_lm_packed_waves == 4) return launch_packed<TM, 1, 4, true, 4>(a, wp, c, M, H, V, groups, s);
    if (groups > 2) return launch_packed<TM, 1, 8, false, 2>(a, wp, c, M, H, V, groups, s);
    if (groups == 1 && g_lm_packed_waves != 8 && few_panels(V)) {
        if (ordinary_stores(H, V)) return launch_packed<TM, 2, 4, false, 2>(a, wp, c, M, H, V, groups, s);
        return launch_packed<TM, 2, 4, true, 2>(a, wp, c, M, H, V, groups, s);
    }
    return launch_packed<TM, 1, 8, true, 2>(a, wp, c, M, H, V, groups, s);
}

template <int TM>
static int launch_rows(const uint16_t* a, const uint16_t* w, float* c, int M, int H, int V, hipStream_t s)
{
    if (few_panels(V)) return launch_packed<TM, 2, 4, true, 2, false, true>(a, w, c, M, H, V, 1, s);
    return launch_packed<TM, 1, 8, true, 2, false, true>(a, w, c, M, H, V, 1, s);
}

// The same kernel on a row-major matrix, for spec_lm_head (M <= 160, H a multiple of 256).  Returns false if it does not take the shape: the 4-wave
// kernel of lm_head.hip, whose passes are half as wide, serves it then.
// That one splits a small vocabulary over more waves, and with few rows over more workgroups.  Measured against it (4-wave -> this, three matrices in
// turn, us):
//   11 panels per CU and more: V = 151936, H = 4096 M = 1 225 -> 203, M = 40 250 -> 222, M = 150 329 -> 299; V = 50021, H = 1280 M = 1 27.8 -> 27.0,
//     M = 150 58 -> 50; V = 42000, H = 2560 M = 1 45.7 -> 44.9, M = 150 75.6 -> 62.1
//   8: V = 32000 M = 1 H = 1024 14.6 -> 14.6, H = 2048 30.9 -> 28.1, H = 4096 62 -> 57, M = 80 17.5 -> 15.8, 36.5 -> 33.5, 64 -> 60
//   9 and 10: V = 36000 M = 12 H = 1280 23.4 -> 23.8, H = 2560 43.8 -> 46.0, H = 4096 76 -> 73, M = 40 26.1 -> 25.4, 49.7 -> 50.5, 82 -> 78, M = 80 32.7 -> 29.7
//   fewer (one matrix): V = 24576, H = 2048 M = 1 18.9 -> 20.3, M = 160 28.9 -> 31.7; V = 16000, H = 1024 8.8 -> 11.6, 17.0 -> 19.0; V = 2000, H = 4096 21.9 -> 33.4
// Reading 64 bytes of each of 16 rows instead (no weaving, ordinary loads) costs the same from M = 96 on, and 222 against 199 us at M = 5.
bool lm_head_rows_dispatch(const uint16_t* a, const uint16_t* w, float* c, int M, int H, int V, hipStream_t s, int* rc)
{
    if (M > kPkMaxRows || H % (2 * kPkSlab) != 0 || (size_t)V > ((size_t)1 << 32) / (4 * (size_t)(kPkMaxRows + 16))) return false;
    const int panels = panels_per_cu(V);
    if (panels < 8 || (panels < 11 && panels > 8 && M <= 32)) return false;
    switch ((M + 15) / 16) {
        case 1: case 2: *rc = launch_rows<2>(a, w, c, M, H, V, s); break;
        case 3: case 4: *rc = launch_rows<4>(a, w, c, M, H, V, s); break;
        case 5: case 6: *rc = launch_rows<6>(a, w, c, M, H, V, s); break;
        case 7: case 8: *rc = launch_rows<8>(a, w, c, M, H, V, s); break;
        default: *rc = launch_rows<10>(a, w, c, M, H, V, s); break;
    }
    return true;
}

}  // namespace specv

extern "C" size_t spec_lm_head_packed_bytes(int V, int H)
{
    if (V <= 0 || H <= 0) return 0;
    return (size_t)((V + 15) / 16) * 16 * (size_t)H * 2;
}

extern "C" int spec_lm_head_pack(const void* W, void* Wp, int V, int H, void* stream)
{
    using namespace specv;
    if (V < 0 || H <= 0) return fail(SPEC_EINVAL, "spec_lm_head_pack: negative size (V=%d H=%d)", V, H);
    if (V == 0) return SPEC_OK;
    if (!W || !Wp) return fail(SPEC_EINVAL, "spec_lm_head_pack: NULL pointer argument");
    if (H % 32 != 0) return fail(SPEC_ESHAPE, "spec_lm_head_pack: H=%d must be a multiple of 32", H);
    if (!aligned(W, 16) || !aligned(Wp, 16)) return fail(SPEC_EINVAL, "spec_lm_head_pack: operands must be 16-byte aligned");
    const size_t n_chunks = spec_lm_head_packed_bytes(V, H) / 16;
    const size_t want = (n_chunks + 255) / 256;
    const unsigned grid = (unsigned)(want < 65536 ? want : 65536);
    hipLaunchKernelGGL(lm_head_pack_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream,
                       (const uint16_t*)W, (uint16_t*)Wp, V, H, n_chunks);
    return check_launch("spec_lm_head_pack");
}

namespace specv {

extern Tunable g_lm_packed_tile;
int lm_head_mfma_dispatch(const uint16_t* a, const uint16_t* wp, float* c, int M, int H, int V, const LmSummary* summary, hipStream_t s);
int lm_head_mfma_blocks(int M, int H, int V);

// (the hooks speak of the weight-streaming kernel)
static bool large_tile_faster(int M, int H, int V)
{
    // (rows first: the number of CUs is a call into the runtime)
    return M > 112 && M <= kPkMaxRows && g_lm_packed_waves == 0 && g_lm_packed_wide != 1 && lm_packed_large_tile(M, H, V, device_cu_count(), kMemorySideCache);
}

static int packed_groups(int M) { return (M + kPkMaxRows - 1) / kPkMaxRows; }

// shared by spec_lm_head_packed (blk_max == nullptr) and spec_lm_head_packed_stats
static int lm_head_packed_any(const char* who, const void* hidden, const void* Wp, float* logits, int M, int H, int V,
                              float* blk_max, int32_t* blk_arg, void* stream, const LmSummary* summary = nullptr)
{
    if (M < 0 || H <= 0 || V < 0) return fail(SPEC_EINVAL, "%s: negative size (M=%d H=%d V=%d)", who, M, H, V);
    if (M == 0 || V == 0) return SPEC_OK;
    if (!hidden || !Wp || !logits) return fail(SPEC_EINVAL, "%s: NULL pointer argument", who);
    if (H % (2 * kPkSlab) != 0) return fail(SPEC_ESHAPE, "%s: H=%d must be a multiple of %d", who, H, 2 * kPkSlab);
    if (!aligned(hidden, 16) || !aligned(Wp, 16) || !aligned(logits, 16))
        return fail(SPEC_EINVAL, "%s: operands must be 16-byte aligned", who);
    if ((size_t)V > ((size_t)1 << 32) / (4 * (size_t)(kPkMaxRows + 16)))
        return fail(SPEC_ESHAPE, "%s: V=%d is beyond the 32-bit row offsets of the kernel", who, V);
    hipStream_t s = (hipStream_t)stream;
    const uint16_t* wp = (const uint16_t*)Wp;
    // More than 160 rows: the contraction is bound by the matrix cores, and the large-tile kernel serves it
    const bool large_tile_fits = (M > kPkMaxRows || (!summary && large_tile_faster(M, H, V))) && (size_t)V <= ((size_t)1 << 32) / (4 * (size_t)(304 + 16));
    if (summary && !large_tile_fits) return fail(SPEC_ESHAPE, "%s: block summaries need more than %d rows (M=%d, V=%d)", who, kPkMaxRows, M, V);
    if (!blk_max && large_tile_fits && (summary || g_lm_packed_tile != 1)) {
        const int rc = lm_head_mfma_dispatch((const uint16_t*)hidden, wp, logits, M, H, V, summary, s);
        if (rc != SPEC_OK) return rc;
        return check_launch(who);
    }
    // More rows than a workgroup holds: the rows are cut into equal groups of at most 160 (a multiple of 16 each), and
    // the grid is groups x panel ranges.  HBM still sees W once; the other groups read it from the L2.
    int groups = packed_groups(M);
    int tm = ((M + groups - 1) / groups + 15) / 16;                     // 16-row tiles per group, 1 .. 10
    const uint16_t* a = (const uint16_t*)hidden;
    int rc;
    // Groups of at most 80 rows leave registers for 4 panels per wave: a pass is 512 entries wide, which halves the LDS
    // reads per MFMA and quarters the re-reads of hidden, at the price of W crossing L2 -> CU twice as often.
    if (!blk_max && g_lm_packed_wide == 1 && g_lm_packed_waves != 4) {
        groups = (M + kPkMaxRows / 2 - 1) / (kPkMaxRows / 2);
        tm = ((M + groups - 1) / groups + 15) / 16;                     // 1 .. 5
        if (groups > 2) rc = launch_packed<5, 1, 8, false, 4>(a, wp, logits, M, H, V, groups, s);
        else if (tm <= 2) rc = launch_packed<2, 1, 8, true, 4>(a, wp, logits, M, H, V, groups, s);
        else if (tm <= 4) rc = launch_packed<4, 1, 8, true, 4>(a, wp, logits, M, H, V, groups, s);
        else rc = launch_packed<5, 1, 8, true, 4>(a, wp, logits, M, H, V, groups, s);
        if (rc != SPEC_OK) return rc;
        return check_launch(who);
    }
    switch (tm) {
        case 1: case 2: rc = launch_packed_auto<2>(a, wp, logits, M, H, V, groups, s, blk_max, blk_arg); break;
        case 3: case 4: rc = launch_packed_auto<4>(a, wp, logits, M, H, V, groups, s, blk_max, blk_arg); break;
        case 5: case 6: rc = launch_packed_auto<6>(a, wp, logits, M, H, V, groups, s, blk_max, blk_arg); break;
        case 7: rc = launch_packed_auto<7>(a, wp, logits, M, H, V, groups, s, blk_max, blk_arg); break;
        case 8: rc = launch_packed_auto<8>(a, wp, logits, M, H, V, groups, s, blk_max, blk_arg); break;
        case 9: rc = launch_packed_auto<9>(a, wp, logits, M, H, V, groups, s, blk_max, blk_arg); break;
        default: rc = launch_packed_auto<10>(a, wp, logits, M, H, V, groups, s, blk_max, blk_arg); break;
    }
    if (rc != SPEC_OK) return rc;
    return check_launch(who);
}

}  // namespace specv

extern "C" int spec_lm_head_packed(const void* hidden, const void* Wp, float* logits, int M, int H, int V, void* stream)
{
    return specv::lm_head_packed_any("spec_lm_head_packed", hidden, Wp, logits, M, H, V, nullptr, nullptr, stream);
}

/* blocks per row of the statistics spec_lm_head_packed_stats writes; 0 = the packed kernel does not take this shape */
extern "C" int spec_lm_head_packed_stats_blocks(int M, int H, int V)
{
    using namespace specv;
    if (M <= 0 || H <= 0 || V <= 0 || H % (2 * kPkSlab) != 0) return 0;
    int ranges, per_range;
    packed_geometry(V, packed_groups(M), &ranges, &per_range);
    return ranges * ((per_range + 15) / 16);
}

/* blocks per row of the summaries spec_lm_head_packed_summary writes; 0 = that call does not take this shape */
extern "C" int spec_lm_head_packed_summary_blocks(int M, int H, int V)
{
    using namespace specv;
    if (M <= kPkMaxRows || (size_t)V > ((size_t)1 << 32) / (4 * (size_t)(304 + 16))) return 0;
    return lm_head_mfma_blocks(M, H, V);
}

extern "C" int spec_lm_head_packed_summary(const void* hidden, const void* Wp, float* logits, int M, int H, int V,
                                           const float* temperature, const int32_t* qo_indptr, int B,
                                           float* blk_max, float* blk_sum, int32_t* blk_span, void* stream)
{
    using namespace specv;
    if (M > 0 && V > 0 && (!temperature || !qo_indptr || B <= 0 || !blk_max || !blk_sum || !blk_span))
        return fail(SPEC_EINVAL, "spec_lm_head_packed_summary: NULL pointer argument or B=%d", B);
    LmSummary sm{};
    sm.temperature = temperature; sm.qo_indptr = qo_indptr; sm.B = B;
    sm.blk_max = blk_max; sm.blk_sum = blk_sum; sm.blk_span = blk_span;
    return lm_head_packed_any("spec_lm_head_packed_summary", hidden, Wp, logits, M, H, V, nullptr, nullptr, stream, &sm);
}

extern "C" int spec_lm_head_packed_stats(const void* hidden, const void* Wp, float* logits, int M, int H, int V,
                                         float* blk_max, int32_t* blk_arg, void* stream)
{
    using namespace specv;
    if (M > 0 && V > 0 && (!blk_max || !blk_arg)) return fail(SPEC_EINVAL, "spec_lm_head_packed_stats: NULL pointer argument");
    return lm_head_packed_any("spec_lm_head_packed_stats", hidden, Wp, logits, M, H, V, blk_max, blk_arg, stream);
}
