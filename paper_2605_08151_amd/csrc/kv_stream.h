// Whether the K/V pages of a chunk are worth nontemporal loads.  Plain arithmetic without device types: the attention kernels and a CPU test
// share it.
//
// A page that one workgroup reads once, in a batch whose K/V does not fit the memory-side cache, is read nontemporal; anything else keeps the
// ordinary loads.  Both conditions are taken from the batch itself, since the bounds a server states may be its model's maximum in every call and a
// page table may map the pages of a common prefix into many requests.  Measured on MI355X, ordinary / nontemporal for all, us per call:
//   64 requests x 8 kv heads x 4.1-4.6k keys (1.1 GB), own pages 206 / 182 (decode), 219 / 206 (5 rows); sharing a prefix of 4096 keys 79 / 96, 98 / 118
//   128 x 8 x 2.0-2.3k keys 198 / 178; sharing 2048 keys 73 / 85
//   64 x 1 x 1-4k keys (83 MB, found in the cache by the next call) 39 / 42; 64 x 8 x 64-256 keys (42 MB) 36.6 / 38.8
#pragma once

#include <cstdint>

namespace specv {

constexpr int kKvScanRequests = 1024;          // at most so many requests around its own are looked at by a workgroup

struct KvScan {
    float keys;                                // committed keys of the requests looked at
    bool shared;                               // another request maps the same page at the same place
};

// Part `part` of `parts` of the scan for request i, whose chunk starts at page index `page`: requests part, part + parts, ... of the window.
constexpr KvScan kv_scan_part(const int32_t* seq_lens, const int32_t* page_table, int max_pages, int B, int max_kv_len, int i, int page, int part, int parts)
{
    KvScan r{0.0f, false};
    int first = i - kKvScanRequests / 2;
    if (first > B - kKvScanRequests) first = B - kKvScanRequests;
    if (first < 0) first = 0;
    const int last = first + kKvScanRequests < B ? first + kKvScanRequests : B;
    const int32_t own = page_table[(long)i * max_pages + page];
    for (int j = first + part; j < last; j += parts) {
        const int c = seq_lens[j];
        const int32_t other = page_table[(long)j * max_pages + page];    // (requested together with the length)
        const int keys = c < 0 ? 0 : (c < max_kv_len ? c : max_kv_len);
        r.keys += (float)keys;
        r.shared |= (j != i) & (other == own) & (page < keys / 16);       // (entries past a request's committed keys may be stale)
    }
    return r;
}

}  // namespace specv
