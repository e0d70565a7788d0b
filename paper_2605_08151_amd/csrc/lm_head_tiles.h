// Row groups, panel ranges and panel shares of the large-tile LM head (lm_head_mfma_kernel.h), and which bytes of the packed matrix a wave
// requests for them.  Integer arithmetic only, without device types: the kernel, its launch and a CPU test that walks whole matrices share it.
#pragma once

#include <cstddef>
#include <cstdint>

namespace specv {

constexpr int kMfWaves = 4;                    // waves per workgroup
constexpr int kMfTN = 4;                       // panels (16 vocabulary entries each) per wave
constexpr int kMfPassPanels = kMfWaves * kMfTN;
constexpr int kMfTallTM = 18;                  // row tiles per group at most

// Row groups, panel ranges and the instantiation that serves them.
struct MfmaLayout { int groups, tiles_lo, groups_hi, tm, ranges, per_range, passes_per_range, blocks; };

// Panels of a range when `groups` row groups share the CUs: as many ranges as there are CUs per group, a multiple of 8 (one per XCD and step of
// the dealing).
constexpr int mf_per_range(int n_panels, int groups, int cus)
{
    const int per_xcd = cus / groups / 8;
    const int r0 = per_xcd > 0 ? per_xcd * 8 : 8;
    return (n_panels + r0 - 1) / r0;
}

// Time of a workgroup in units of half a row tile's products for one panel per wave: a pass costs as many panel slots as its fullest wave owns
// (two at least), each 2 tm + 11 (the products, and the operands and the epilogue that do not depend on the rows).  It chooses among groups of up to 16 tiles, and was fitted when all passes
// went through the code for four panels per wave; a last pass with up to two now costs 0.73 of a full one (mf_slots10), not the half that stands here.
constexpr long mf_group_cost(int tiles, int groups, int n_panels, int cus)
{
    const int per_range = mf_per_range(n_panels, groups, cus), tm = (tiles + groups - 1) / groups;
    const int rest = per_range % kMfPassPanels, last = (rest + kMfWaves - 1) / kMfWaves;
    const long slots = (long)(per_range / kMfPassPanels) * kMfTN + (rest == 0 ? 0 : (last > 2 ? last : 2));
    return slots * (2 * tm + 11);
}

constexpr MfmaLayout mf_layout_of(int tiles, int groups, int n_panels, int cus)
{
    MfmaLayout L{};
    L.groups = groups;
    L.tiles_lo = tiles / groups;                                         // groups of tiles_lo + 1 first, then of tiles_lo
    L.groups_hi = tiles % groups;
    L.tm = L.tiles_lo + (L.groups_hi ? 1 : 0);
    L.per_range = mf_per_range(n_panels, groups, cus);
    L.ranges = ((n_panels + L.per_range - 1) / L.per_range + 7) / 8 * 8;
    L.passes_per_range = (L.per_range + kMfPassPanels - 1) / kMfPassPanels;
    L.blocks = L.ranges * L.passes_per_range * kMfWaves;
    return L;
}

// cap_rows: rows per group at most (144..256); anything else = automatic.
constexpr MfmaLayout mfma_layout_for(int M, int V, int cus, int cap_rows)
{
    constexpr int kMinTM = 9, kMaxTM = 16;                               // the kernel is built for 9..16 tiles per group
    const int tiles = (M + 15) / 16;                                     // 16-row tiles of the batch
    const int n_panels = (V + 15) / 16;
    const bool forced = cap_rows >= 16 * kMinTM && cap_rows <= 16 * kMaxTM;
    const int cap_tiles = forced ? cap_rows / 16 : kMaxTM;
    int groups = (tiles + cap_tiles - 1) / cap_tiles;
    while (groups > 1 && (tiles + groups - 1) / groups < kMinTM) --groups;
    // As few groups as 16 tiles each allow: the taller the tile, the fewer bytes go from L2 to the CUs per product.  Measured on MI355X
    // (V = 151936, H = 4096), groups of at most 13 / at most 16 tiles: M = 480 576 / 506 us, M = 768 788 / 773, M = 1024 1035 / 1004,
    // M = 1152 1164 / 1151.  One or two more where that leaves the last pass of every range, or CUs, much emptier: 3 / 4 groups at V = 32000,
    // H = 4096 (25 panels a range, 16 + 9 / 32): M = 640 166 / 137 us, M = 768 190 / 154; V = 64000, H = 1280: M = 704 137 / 126.
    if (!forced) {
        long best = mf_group_cost(tiles, groups, n_panels, cus) * 97 / 100;
        const int fewest = groups;
        for (int g = fewest + 1; g <= fewest + 2 && (tiles + g - 1) / g >= kMinTM; ++g) {
            const long cost = mf_group_cost(tiles, g, n_panels, cus);
            if (cost < best) { best = cost; groups = g; }
        }
    }
    return mf_layout_of(tiles, groups, n_panels, cus);
}

// The same for groups of 17 or 18 tiles, which take fewer bytes from L2 per product and, where they make the number of groups a power of two, leave no CU
// idle (3 groups of 12 and 5 of 15 occupy 240 of 256); groups == 0: up to 16 tiles it is.
// By tenths of a panel slot: a last pass with two panels per wave costs 0.73 of a full one, with three 0.87 (all of it beyond 16 tiles, where the code for four
// serves it).  Measured, at most 16 / 17 and 18 tiles, us: H = 4096 V = 151936 M = 272 344 / 322, M = 544 595 / 561, M = 576 606 / 586, M = 800 815 / 796,
// M = 1056 1070 / 1021, M = 1152 1148 / 1097; V = 128256 M = 288 301 / 268, M = 576 540 / 476, M = 1152 987 / 909; V = 32000 M = 576 138 / 127, M = 1152 261 / 235;
// H = 2560 V = 64000 M = 272 98 / 90, M = 576 184 / 162.  Not chosen: H = 4096 V = 100000 M = 576 403 / 419 (3 full passes and one panel),
// V = 128256 M = 800 678 / 689; H = 1024 V = 32000 M = 288 25 / 28.5.
constexpr long mf_slots10(int per_range, int tm)
{
    const int rest = per_range % kMfPassPanels, last = (rest + kMfWaves - 1) / kMfWaves;
    return (long)(per_range / kMfPassPanels) * 40 + (rest == 0 ? 0 : last <= 2 ? 29 : (last == 3 && tm <= 16) ? 35 : 40);
}

constexpr long mf_tall_cost(int tiles, int groups, int n_panels, int cus)
{
    const int per_range = mf_per_range(n_panels, groups, cus), tm = (tiles + groups - 1) / groups;
    return mf_slots10(per_range, tm) * (2 * tm + 6);
}

constexpr MfmaLayout mfma_tall_layout_for(int M, int V, int cus)
{
    const int tiles = (M + 15) / 16, n_panels = (V + 15) / 16;
    long best = mf_tall_cost(tiles, mfma_layout_for(M, V, cus, 0).groups, n_panels, cus);
    int groups = 0;
    for (int g = (tiles + kMfTallTM - 1) / kMfTallTM; (tiles + g - 1) / g > 16; ++g) {
        const long cost = mf_tall_cost(tiles, g, n_panels, cus);
        if (cost < best) { best = cost; groups = g; }
    }
    return groups == 0 ? MfmaLayout{} : mf_layout_of(tiles, groups, n_panels, cus);
}

// Whether the products weigh enough for them: what a tile costs besides (its operands' first slabs, its stores) grows with its height.  At most 16 / 17 and 18 tiles, us, one group: H = 256 V = 64000
// M = 260 19.4 / 22.2, V = 128256 M = 288 39 / 43; H = 512 V = 128256 60 / 64, V = 100000 55.6 / 52.2; H = 768 V = 50021 34.3 / 32.8, V = 128256 79 / 76, V = 64000 35.5 / 36.7.
// Several groups: H = 256 V = 32000 M = 560, one pass, 19.8 / 21.0, V = 64000, two, 44.6 / 36.1, V = 128256 M = 1152 191 / 146; H = 512 V = 32000 M = 560 29.5 / 29.8, M = 1152 53 / 51.
constexpr bool mfma_tall_pays(const MfmaLayout& L, int H)
{
    return L.groups == 1 ? H >= 768 : H >= 512 || L.per_range > kMfPassPanels;
}

// How W is read: buffer loads; global loads; nontemporal global loads; the same two of a matrix that is row-major, not packed
enum MfmaLoads { kBufferLoads, kGlobalLoads, kStreamLoads, kRowLoads, kRowStreamLoads };

// One row group reads W once, bound by that stream: nontemporal, by the rule of the weight-streaming kernel (the tree step, M = 188, V = 151936,
// H = 4096 378 -> 360 us, M = 216 408 -> 394; V = 64000, H = 2560 179 -> 167).
// Several groups that read panels a multiple of 64 KB apart: global loads (buffer -> global, V = 151936 / 100000, H = 4096: M = 257 357 -> 330 /
// 264 -> 247 us, M = 576 622 -> 606 / 408 -> 395, M = 1152 1157 -> 1119 / 793 -> 782; H = 2048 M = 257 191 -> 179, M = 576 351 -> 328).  Elsewhere
// buffer loads (H = 2560: M = 576 398 -> 409 / 260 -> 265, M = 1152 757 -> 779; H = 3072 854 -> 902; H = 1024 357 -> 360).
constexpr MfmaLoads mfma_loads_for(int groups, int H, int V, size_t cache = (size_t)256 << 20)
{
    if (groups == 1 && (size_t)V * H * 2 > cache * 3 / 8) return kStreamLoads;
    return groups > 1 && H % 2048 == 0 ? kGlobalLoads : kBufferLoads;
}

// The instantiations of lm_head_tile.hip; lm_head_mfma_buffer.hip and _global.hip have 9 to 16 row tiles, _stream.hip 11 to 16.
constexpr bool mf_tile_built(MfmaLoads loads, int tm)
{
    if (loads > kStreamLoads) return false;
    return tm == 17 || tm == 18 || (tm == 8 && loads != kGlobalLoads) || ((tm == 9 || tm == 10) && loads == kStreamLoads);
}

// Between 113 and 160 rows (8 to 10 row tiles) the large-tile kernel is ahead where the products weigh: it reads a fragment of hidden from LDS for 4 panels,
// not for 2, stages hidden without registers and requests 2.5 to 4 slabs ahead.  The weight-streaming kernel (lm_head_packed.hip) is ahead (or as fast) where all its waves have
// their two panels in one pass, 13 to 16 panels per CU, with aligned stores; and with few rows or short ones on a small matrix.  Measured, weight-streaming -> large tile, us:
//   17 panels per CU and more: V = 151936, H = 4096 M = 113 224 -> 211, M = 128 230 -> 214, M = 144 248 -> 221, M = 160 260 -> 224; V = 100000 M = 160 172 -> 153;
//     V = 68000, H = 1280 M = 120 55.1 -> 49.7, M = 160 60.8 -> 54.6; V = 131072, H = 1024 M = 128 64.8 -> 65.0, M = 160 69.5 -> 68.8
//   13 to 16: V = 64000, H = 2560 M = 113 61.4 -> 62.9, M = 160 64.6 -> 68.4; V = 57344, H = 1280 M = 160 37.9 -> 41.1 (but H = 4096 96.3 -> 90.9: left as it was);
//     but rows of logits that are not aligned V = 64013, H = 2560 M = 128 69 -> 66, M = 160 76 -> 69, V = 57345, H = 1280 40.1 -> 36.4, 45.7 -> 40.0
//   10 to 12: V = 49152 M = 128 H = 1280 32.8 -> 31.1, H = 4096 79 -> 72; V = 40000, H = 1024 M = 128 19.7 -> 19.2; but H = 512 V = 40000 M = 128 13.2 -> 13.8, M = 160 15.7 -> 14.9 and 16.1 -> 19.6,
//     V = 44000 M = 128 13.8 -> 15.0, M = 144 15.0 -> 15.8
//   9: V = 36864 M = 128 H = 2048 39.6 -> 37.0, but H = 1280 (94 MB, ordinary loads) 23.0 -> 25.9
//   5 to 8: V = 32000, H = 1024 M = 128 19.7 -> 19.8, M = 160 21.3 -> 20.8, H = 2560 35.8 -> 37.9, 40.8 -> 39.8, H = 4096 52 -> 50 (M = 128: left as it was), 62 -> 53
//   fewer: V = 16000, H = 2048 M = 128 25.8 -> 19.4, H = 256 6.7 -> 6.2; V = 2000, H = 4096 M = 160 46 -> 30, but H = 256 M = 144 6.7 -> 7.0; V = 12000, H = 256 7.0 -> 7.3
constexpr bool lm_packed_large_tile(int M, int H, int V, int cus, size_t cache = (size_t)256 << 20)
{
    if (M <= 112 || M > 160) return false;
    if (V % 4 != 0) return true;
    const int panels = mf_per_range((V + 15) / 16, 1, cus);
    if (panels > 16) return true;
    if (panels > 12) return false;
    if (panels >= 10) return H >= 1024;
    if (panels == 9) return (size_t)V * H * 2 > cache * 3 / 8;
    if (panels >= 5) return M > 128;
    return H >= 512 || panels == 4;
}

// Rows of a tile of the kernel with 32 x 32 products (lm_head_big2_kernel), whichever of the two pads less; a tile is 256 vocabulary entries wide.
constexpr int lm_big2_rows(int M) { return (M + 191) / 192 * 192 <= (M + 255) / 256 * 256 ? 192 : 256; }

// Whether row-major weights go through the large-tile kernel.  More than 160 rows, against the kernel with 32 x 32 products, us:
//   one row group: V = 151936, H = 4096 M = 192 371 -> 296; V = 64000, H = 2560 M = 200 99 -> 86; V = 32000, H = 4096 M = 256 112 -> 84; V = 2000, H = 2048 M = 224 52 -> 32;
//     13 to 15 panels per CU, one pass that wastes slots, only where the other one pads the rows (193 to 224) or W's stream weighs: V = 50021, H = 2048 M = 177 58 -> 63, M = 208 69 -> 67,
//     M = 256 70 -> 75, H = 4096 118 -> 114, 133 -> 121, 135 -> 136; V = 57344, H = 1024 M = 177 32.0 -> 36.6.
//     H = 256, up to 192 rows: V = 4000 M = 177 9.7 -> 10.8, V = 12001 10.8 -> 12.3, V = 40001 13.9 -> 14.6; but V = 24000 12.0 -> 11.5, V = 151936 44 -> 35
//   several: by the time of a workgroup's tiles, the rounds of the other kernel's tiles over the CUs times their rows against the panel slots of a range times 2 tm + 11 (see
//     mf_group_cost).  Per unit this kernel is the faster one by 0.64 (0.69 where rows are no power of two apart: the other one reads those faster; 0.62 either way from 1 GiB of W on:
//     V = 151936 M = 576 H = 4096 793 -> 741, H = 6144 1169 -> 1125, H = 8192 1521 -> 1409, M = 1152 H = 6144 2173 -> 2061).  Taken:
//     V = 151936, H = 4096 M = 320 536 -> 451, M = 1152 1489 -> 1368; V = 50021, H = 2560 M = 768 249 -> 204.  Not taken: M = 576 V = 64000, H = 2560 212 -> 258, V = 128256,
//     H = 2560 414 -> 475, V = 151936, H = 2048 414 -> 431; M = 1152 V = 64000, H = 2048 332 -> 349, V = 100000, H = 3072 765 -> 798.  Of 800 shapes of H = 1024 to 8192, M = 257 to
//     4096, V = 8001 to 151936 the slower one is taken by more than 2 % in 33, by 6 % at most (five groups on 240 of 256 CUs above all).
//     H = 256, where a range is one pass with three or four panels per wave and the other kernel one round: V = 28002 M = 300 14.3 -> 16.1, V = 8000 M = 1152 13.6 -> 15.2
// 113 to 160 rows, against the weight-streaming kernels, by panels per CU:
//   17 and more: V = 151936 M = 128 H = 4096 284 -> 249, H = 1280 107 -> 99.5; V = 128256, H = 2048 135 -> 133; V = 68000, H = 2560 113 -> 103
//   13 to 16: V = 64000, H = 2560 M = 128 70 -> 73; rows of logits not aligned V = 61001, H = 2048 M = 128 65.7 -> 60.8, M = 160 72.7 -> 63.9, V = 53249, H = 4096 108.5 -> 109.3
//   9 to 12: V = 36864 M = 128 H = 1280 32.9 -> 30.1, H = 4096 89 -> 79; V = 45056, H = 1280 33.6 -> 33.7; V = 49152, H = 2048 55.7 -> 54.3
//   8: V = 32000 M = 128 H = 1024 17.0 -> 17.9, H = 4096 64.8 -> 64.7; V = 32001, H = 2560 44.1 -> 49.1
//   fewer, aligned: not measured, as 8; not aligned V = 24001, H = 1280 M = 128 24.6 -> 22.3, V = 20001, H = 2048 M = 160 34.7 -> 32.0, V = 8001, H = 4096 34.5 -> 45; but not where this
//     kernel reads W nontemporal and the memory-side cache holds much of it from one call to the next (over three matrices in turn V = 24001, H = 2560, 117 MiB, M = 128 41.7 -> 44.5; two in
//     turn V = 20001, H = 4096, 156 MiB 52.9 -> 54.9, V = 24001, H = 4096, 188 MiB 58.6 -> 57.8, V = 28001, 219 MiB 64 -> 61)
constexpr bool lm_rowmajor_large_tile(int M, int H, int V, int cus, size_t cache = (size_t)256 << 20)
{
    if (M <= 112 || H % 256 != 0 || (size_t)V > ((size_t)1 << 32) / (4 * (size_t)(304 + 16))) return false;
    const int n_panels = (V + 15) / 16, panels = mf_per_range(n_panels, 1, cus);
    if (M <= 160) {
        if (panels < 5 || panels == 8 || (V % 4 == 0 && (panels < 8 || (panels > 12 && panels <= 16)))) return false;
        const size_t bytes = (size_t)V * H * 2;
        return panels > 8 || bytes <= cache * 3 / 8 || bytes > cache * 5 / 8;
    }
    const MfmaLayout L = mfma_layout_for(M, V, cus, 0);
    if (L.groups == 1) {
        if (panels >= 13 && panels <= 15 && H < 4096) return M > 192 && M <= 224;
        return H >= 512 || M > 192 || (panels >= 6 && panels <= 8) || panels > 16;
    }
    const int rows = lm_big2_rows(M);
    const long tiles = (long)((M + rows - 1) / rows) * ((V + 255) / 256), rounds = (tiles + cus - 1) / cus;
    if (H < 512 && rounds == 1 && L.per_range > 10 && L.per_range <= kMfPassPanels) return false;
    const int per_unit = (size_t)V * H * 2 >= cache * 4 ? 619 : (H & (H - 1)) == 0 ? 642 : 692;
    return rounds * rows * 5000 >= per_unit * mf_slots10(L.per_range, L.tm) * (2 * L.tm + 11);
}

struct PanelShare { int p0, np; };             // first panel and number of panels, 0 .. 4; p0 is a panel of the range also where np == 0

// What wave `wave` owns in pass `pass` of the range [p_begin, p_end): passes are full (16 panels, 4 per wave) up to the last, which deals
// its 1..16 panels as evenly as they go.
constexpr PanelShare mf_panel_share(int p_begin, int p_end, int pass, int wave)
{
    const int lo = p_begin + pass * kMfPassPanels;
    const int m = p_end - lo < kMfPassPanels ? p_end - lo : kMfPassPanels;
    const int first = wave * m / kMfWaves;
    return {lo + first, (wave + 1) * m / kMfWaves - first};
}

// Passes of the range with 16 panels, all their entries in the matrix: all, where the panels divide and the last one is not padded, else all but the
// last.
constexpr int mf_full_passes(int p_begin, int p_end, int V)
{
    return (p_end - p_begin - (p_end * 16 > V ? 1 : 0)) / kMfPassPanels;
}

// Panels per wave that the code of a range's last pass serves: 2, 3 or 4 (one panel in code for one would not be faster: the pass is bound by
// the fragments of hidden that every wave reads from LDS).
constexpr int mf_last_slots(int n_own)
{
    const int m = (n_own - 1) % kMfPassPanels + 1, most = (m + kMfWaves - 1) / kMfWaves;
    return most < 2 ? 2 : most;
}

// Byte distance of panel slot tn from the wave's first panel.  A slot past the wave's share repeats its last panel (the L2 or the
// L1 has it, its products are never stored), so that every request lies inside the matrix by its address alone: a buffer
// descriptor's bounds check does not cover the scalar offset.
constexpr uint32_t mf_slot_bytes(int np, int tn, uint32_t panel_bytes)
{
    const int last = np > 0 ? np - 1 : 0;
    return (uint32_t)(tn < last ? tn : last) * panel_bytes;
}

}  // namespace specv
