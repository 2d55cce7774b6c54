// How many LDS buckets the records and the dedup take, and whether they can: host arithmetic
// without a device, so that a test can walk all of it.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace mj {

constexpr int BK_AVG = 1024;    // records of a bucket aimed at (keys are hashes)
constexpr int BK_AVG_MEMBERS = 384;  // where (nearly) all of them are members: half of BK_CAP
constexpr int BK_CAP = 768;     // members of a bucket in short slots
constexpr int BK_BITS_MAX = 16; // bucket bits (two radix passes)

constexpr int DD_CAP = 4096, DD_LOG = 13, DD_AVG = 3072, DD_PARTS = 12;
constexpr int DD_BITS_MAX = 14;  // bucket bits
constexpr int DD_BATCH = 8;      // loads of a thread in flight
constexpr int64_t DD_SWEEP = 1 << 20;  // of 1.5 M pairs of texts one bucket has 0.5 M candidates: with
                                       // 2^18 that join took 7.70 ms, 7.28 with these

inline int bits_for(int64_t n, int64_t avg) {  // 2^bits buckets of about avg
    int b = 0;
    while (((n + avg - 1) / avg) > (1ll << b)) b++;
    return b;
}

// Bucket bits of `expect` records; small: of buckets of BK_AVG_MEMBERS.
inline int record_bits(int64_t expect, bool small) {
    return std::min(BK_BITS_MAX, bits_for(std::max<int64_t>(expect, 1), small ? BK_AVG_MEMBERS : BK_AVG));
}

// Whether records of which this many share their key want the small buckets (now: have them).  A
// bucket of 512 to 1,024 records holds about members / 2^bits members, and what its LDS holds (768)
// has to be some deviations more, since the members come in groups (of ten: a deviation is 3
// sqrt(members)): 485 K records, all members, in buckets of 947 took the general path after the
// buckets' (candidates 0.85 ms, 0.77 without trying them), in smaller buckets 0.68.  The lower limit
// keeps the choice from swinging.
inline bool small_buckets_pay(int64_t records, int64_t members, bool now) {
    return members >> record_bits(records, false) > (now ? 300 : 560);
}

// Radix passes by the top bits that put the elements of a bucket together: none for one
// bucket, one for up to 2^8, two for up to 2^16.
inline int bucket_passes(int bits) { return bits == 0 ? 0 : bits <= 8 ? 1 : 2; }

inline int id_bits(int32_t count) {
    int b = 0;
    while (b < 32 && (1ull << b) < (uint64_t)std::max(count, 1)) b++;
    return b;
}

// Pairs (first, second) of n_first and n_second strings as keys of kb bits, of which the top
// `bits` number the bucket; expect pairs come, about `distinct` (0: not known) different ones.
// More buckets than keys do not fit: the pairs are then mostly duplicates of a few, which the sort
// of kb bits (one or two passes) spreads over the device and buckets would not.  A bucket's table
// holds the other kb - bits <= 31 bits.
struct DedupPlan {
    int bs, kb, bits;
    bool fits;
};
inline DedupPlan dedup_plan(int64_t expect, int64_t distinct, int32_t n_first, int32_t n_second) {
    DedupPlan p;
    p.bs = id_bits(n_second);
    p.kb = id_bits(n_first) + p.bs;
    p.bits = expect <= DD_CAP * 3 / 4 ? 0 : bits_for(expect, DD_AVG);
    p.fits = p.bits <= DD_BITS_MAX && p.bits <= p.kb && p.kb - p.bits <= 31;
    // The lesser of two strings' ids is not evenly spread, and a bucket of more than DD_CAP distinct
    // pairs goes by parts: half as many different pairs a bucket, or as many as one radix pass
    // still makes (568 K pairs of 24,661 strings, hardly any twice: 0.20 -> 0.13 ms, 0.14 by the sort;
    // 60 K of 8,000: 0.15 -> 0.09).  Halving them for duplicates too does not pay (protein, 10 M of
    // 1.3 M: 0.31 -> 0.36 ms; long DNA, a second pass: 0.06 -> 0.08).
    const int fine = std::max(std::min(8, bits_for(expect, DD_AVG / 2)), bits_for(2 * distinct, DD_AVG));
    if (p.fits && p.bits > 0 && p.bits < fine) p.bits = std::min(std::min(fine, DD_BITS_MAX), p.kb);
    return p;
}

}  // namespace mj
