// Where the attention kernels keep a chunk's page ids, the candidates' parents and the rows' masks in LDS.  Plain arithmetic without device types: kernels, launches and a CPU
// test share it.
#pragma once

namespace specv {

constexpr int kAttnParents = 64;               // a tree has at most so many rows

// 4-byte slots for the page ids of a chunk of `chunk_keys` keys (16 per page): one more than its pages, and an even number, since the parents that follow fill a
// multiple of 8 bytes and the 64-bit masks behind them are read and written whole.
constexpr int attn_page_slots(int chunk_keys) { return (chunk_keys / 16 + 2) & ~1; }

// byte offset of the masks from the page ids
constexpr int attn_mask_offset(int chunk_keys) { return (attn_page_slots(chunk_keys) + kAttnParents) * 4; }

}  // namespace specv
