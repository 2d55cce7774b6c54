// How many LDS buckets a dedup takes, and whether it can: host arithmetic without a device, so
// that a test can walk all of it.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace mj {

constexpr int DD_CAP = 4096, DD_LOG = 13, DD_AVG = 3072, DD_PARTS = 12;
constexpr int DD_BITS_MAX = 14;  // bucket bits
constexpr int DD_BATCH = 8;      // loads of a thread in flight
constexpr int64_t DD_SWEEP = 1 << 20;

inline int bits_for(int64_t n, int64_t avg) {  // 2^bits buckets of about avg
    int b = 0;
    while (((n + avg - 1) / avg) > (1ll << b)) b++;
    return b;
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
// `bits` number the bucket; expect pairs come, duplicates among them.  More buckets than keys
// do not fit: the pairs are then mostly duplicates of a few, which the sort of kb bits (one or
// two passes) spreads over the device and buckets would not.  A bucket's table holds the other
// kb - bits <= 31 bits.
struct DedupPlan {
    int bs, kb, bits;
    bool fits;
};
inline DedupPlan dedup_plan(int64_t expect, int32_t n_first, int32_t n_second) {
    DedupPlan p;
    p.bs = id_bits(n_second);
    p.kb = id_bits(n_first) + p.bs;
    p.bits = expect <= DD_CAP * 3 / 4 ? 0 : bits_for(expect, DD_AVG);
    p.fits = p.bits <= DD_BITS_MAX && p.bits <= p.kb && p.kb - p.bits <= 31;
    return p;
}

}  // namespace mj
