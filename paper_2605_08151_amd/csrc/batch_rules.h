// Rules on the number of requests in a batch.  Plain arithmetic without device types: the launches, their kernels and a CPU test share it.
#pragma once

namespace specv {

// Threads per pair of sequences in divergence_kernel, and positions per thread in one memory round trip.  Few pairs wait for round trips: many positions in each.
// With more pairs than CUs they hide each other's waits, and what counts is what is read for nothing behind an early difference.  Pairs of 3000 tokens that
// differ at 10 / 600 / 2999, and of 16000 at the end, us, in the order 512 x 8, 512 x 2, 256 x 4 (one position of 256 threads before):
//   B = 128 3.3 / 3.3 / 3.2, 13.9 (4.1 / 4.8 / 6.5, 37.9); 256 3.9 / 3.9 / 3.9, 13.8 against 2.7 / 2.6 / 4.6, 17.9
//   B = 384 4.5 / 4.5 / 4.5, 15.7 against 2.8 / 2.8 / 5.1, 19.9; 1024 6.5 / 6.5 / 6.4 against 3.6 / 3.6 / 6.6, 31 against 3.8 / 3.8 / 7.8, 44 (5.4 / 5.7 / 9.8, 55)
//   B = 2048 6.0 / 6.0 / 11.2, 60 against 5.2 / 5.2 / 9.9, 54 (7.9 / 8.0 / 11.1, 63); 8192 46.6 / 46.5 / 46.2 against 15.6 / 15.8 / 43.5 (23 / 25 / 51)
struct DivergenceShape { int threads, per; };
// (256 CUs taken for granted: asking the runtime for the device would cost as much as the rule gives)
constexpr DivergenceShape divergence_shape(int B)
{
    return B <= 256 ? DivergenceShape{512, 8} : B <= 4 * 256 ? DivergenceShape{512, 2} : DivergenceShape{256, 4};
}

// Up to so many requests attention's merge kernels count those that start before their row, 256 in a round trip; beyond, a binary search is ahead, whose dependent
// round trips other workgroups hide, and which reads few bytes.  Requests of one row that are split by their bound, 8 heads, whole call, us, count -> search:
// B = 2048 83 -> 82, 4096 169 -> 159, 8192 365 -> 320, 16384 820 -> 630, 65535 5715 -> 2605; of two rows, 32 heads: 2048 352 -> 343, 4096 759 -> 686, 8192 1770 -> 1439.
// At B = 1024 43 with either.
constexpr int kMergeCounted = 1024;

}  // namespace specv
