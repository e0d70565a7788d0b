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

constexpr int kKvScanRequests = 64;            // at most so many requests around its own are looked at by a workgroup: one per lane of a wave

struct KvScan {
    float keys;                                // committed keys of the request looked at, times the requests each one looked at stands for
    bool shared;                               // it maps the same page at the same place
};

// What lane `lane` looks at for request i, whose chunk starts at page index `page`.
constexpr KvScan kv_scan_lane(const int32_t* seq_lens, const int32_t* page_table, int max_pages, int B, int max_kv_len, int i, int page, int lane)
{
    const int looked_at = B < kKvScanRequests ? B : kKvScanRequests;
    int first = i - kKvScanRequests / 2;
    if (first > B - looked_at) first = B - looked_at;
    if (first < 0) first = 0;
    if (lane >= looked_at) return {0.0f, false};
    const int j = first + lane;
    const int32_t own = page_table[(long)i * max_pages + page], other = page_table[(long)j * max_pages + page];
    const int c = seq_lens[j];
    const int keys = c < 0 ? 0 : (c < max_kv_len ? c : max_kv_len);
    // (entries past a request's committed keys may be stale)
    return {(float)keys * ((float)B / (float)looked_at), j != i && other == own && page < keys / 16};
}

}  // namespace specv
