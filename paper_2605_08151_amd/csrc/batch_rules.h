// Rules on the number of requests in a batch.  Plain arithmetic without device types: the launches, their kernels and a CPU test share it.
#pragma once

#include <cstdint>

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

// Attention in fixed chunks: a request has `splits` places of Hkv workgroups in the grid, by the stated bound, and as many pieces as it is long; what is left over ends at once.
// Workgroups go round the 8 XCDs in grid order, and inside an XCD round its 4 shader engines.  With piece k in place k of every request and Hkv * splits a multiple of a power of two,
// requests that fill only their first places lie on the same ones (4 kv heads, 2 places, 1 piece: all work on four XCDs).  So the pieces of a request begin `turn` places
// on, one more with every group of requests that fills a multiple of 32 workgroups.  Only where a request's places are at most 32 workgroups: with more there was as much
// lost as gained (1550 shapes, lengths that differ or half the bound: 28 faster by more than 3 %, 26 slower); up to 32, of 4700 such shapes 1207 faster, 69 slower.
// Pieces first in the grid -> heads first -> heads first with the turn, us, contexts of half the bound: 128 requests of 5 rows, 2855 keys, 4 heads 167 -> 197 -> 121; 510 of 1 row,
// 2317 keys, 4 heads 553 -> 622 -> 394; 31 of 1 row, 6512 keys, 2 heads 52 -> 59 -> 44.  Pieces first is still ahead by more than 3 % in 20 of 7800: few requests whose
// pieces, about one per CU, meet on one shader engine (9 requests x 2 heads, 9 of 17 places: 64 -> 98).
struct PieceTurn { int shift; uint32_t magic; };

constexpr PieceTurn piece_turn(int Hkv, int splits)
{
    long unit = (long)Hkv * splits;
    if (splits < 2 || unit > 32) return {31, 0};          // no turn: request numbers are below 65536
    int shift = 5;                                        // log2(32 / gcd(32, Hkv * splits))
    for (; unit % 2 == 0; unit /= 2) --shift;
    return {shift, (uint32_t)(0x100000000ull / (uint32_t)splits) + 1};
}

// The piece at place `place` of request i.  (x mod splits by a multiplication: exact for x below 2^16 and splits up to 32, since x * (magic * splits - 2^32) < 2^32.)
constexpr int piece_of_place(PieceTurn t, int splits, int place, int i)
{
    const uint32_t x = (uint32_t)i >> t.shift;
    const int turn = (int)(x - (uint32_t)((uint64_t)x * t.magic >> 32) * (uint32_t)splits);
    const int piece = place - turn;
    return piece < 0 ? piece + splits : piece;
}

}  // namespace specv
