// Shared pieces of the verification kernels.
#pragma once

#include "mj_common.h"

namespace mj {

// The verifiers read strings through their bit planes only (never the input symbols).
struct VSet {
    int32_t n;
    const int64_t *off;
    const int32_t *len;
    const int32_t *kk;
    const uint32_t *planes;
};

// The NP bit planes are interleaved: word w of plane p is planes[w * NP + p], so the planes
// of 32 consecutive symbols share a cache line.  `plane` points at plane p's first word
// (planes + p); returns 32 symbols' bits starting at global bit position bitpos (>= 0).
template <int NP>
__device__ __forceinline__ uint32_t load_word(const uint32_t *plane, int64_t bitpos) {
    int64_t w = bitpos >> 5;
    uint32_t sh = (uint32_t)(bitpos & 31);
    uint32_t lo = plane[w * NP], hi = plane[(w + 1) * NP];
    return __builtin_amdgcn_alignbit(hi, lo, sh);
}

// a & ~(b ^ c): the bits of a where b and c agree, in one v_bitop3 (truth table indexed
// by a << 2 | b << 1 | c: set at 100b and 111b).  With b a plane word of the pattern and c
// a text symbol's plane bit broadcast to all 32 lanes of the word, it narrows a match mask
// to the rows whose plane bit equals the text's.
__device__ __forceinline__ uint32_t and_xnor(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x90);
}

// As load_word, for a string read in either direction.
template <int NP>
__device__ __forceinline__ uint32_t load_dir(const uint32_t *plane, int64_t bitpos, bool rev) {
    // forward: symbols bitpos .. bitpos + 31 at bits 0 .. 31; reversed: bit t holds symbol
    // bitpos + 31 - t.  Positions before the start of the planes read as 0.
    uint32_t w;
    if (bitpos >= 0) w = load_word<NP>(plane, bitpos);
    else if (bitpos > -32) w = load_word<NP>(plane, 0) << (uint32_t)(-bitpos);
    else w = 0u;
    return rev ? __builtin_bitreverse32(w) : w;
}

// The same for all planes at once, without branches: the 2 NP words are adjacent.  (bitpos may
// lie before the planes; what a string's own symbols do not fill is then made up.)
template <int NP>
__device__ __forceinline__ void load_planes(const uint32_t *planes, int64_t bitpos, bool rev,
                                            uint32_t (&out)[NP]) {
    const int64_t at = bitpos < 0 ? 0 : bitpos;
    const uint32_t gap = (uint32_t)min<int64_t>(at - bitpos, 31), sh = (uint32_t)at & 31u;
    const uint32_t *w = planes + (at >> 5) * NP;
    uint32_t v[2 * NP];
#pragma unroll
    for (int p = 0; p < 2 * NP; p++) v[p] = w[p];
#pragma unroll
    for (int p = 0; p < NP; p++) {
        const uint32_t x = __builtin_amdgcn_alignbit(v[NP + p], v[p], sh) << gap;
        out[p] = rev ? __builtin_bitreverse32(x) : x;
    }
}

// The work queue of a persistent launch: interleaved sub-queues, each counter on lines of
// its own.
constexpr int QUEUES = 32;
constexpr int QSTRIDE = 32;  // uint64 words between two sub-queue counters (256 bytes)

// The next pairs (their ranks in the order) for the lanes that ask, -1 where there is none
// left; whole wave.  qj: the wave's current sub-queue; done is set once every sub-queue is dry.
// A wave that finds its sub-queue dry reads all counters and goes on where there are pairs.
// (Trying the sub-queues one by one, one a block of columns, every wave ended with up to 32
// blocks of idle columns and an atomic each: 75 us of a launch, whatever its pairs.)
__device__ __forceinline__ long long take_pairs(unsigned long long *next, int64_t n, bool ask,
                                                int &qj, bool &done) {
    const int lane = threadIdx.x & 63;
    long long got = -1;
    for (uint64_t req = __ballot(ask); req && !done; req = __ballot(ask && got < 0)) {
        const int first = __ffsll((unsigned long long)req) - 1;
        const long long size = n > qj ? (n - qj + QUEUES - 1) / QUEUES : 0;
        const long long want = __popcll(req);
        unsigned long long base = 0;
        if (lane == first) base = atomicAdd(next + qj * QSTRIDE, (unsigned long long)want);
        // (wave-uniform, in scalar registers: a few vector registers more and the kernels' 4
        // waves a SIMD become 3)
        const uint32_t blo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, first);
        const uint32_t bhi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(base >> 32), first);
        const long long b0 = (long long)(((uint64_t)bhi << 32) | blo);
        const long long room = size - b0;  // pairs left here, for the first askers
        const int rank = __popcll(req & ((1ull << lane) - 1));
        if (ask && got < 0 && rank < room) got = (b0 + rank) * QUEUES + qj;
        if (want <= room) break;
        long long left = 0;
        if (lane < QUEUES && n > lane)
            left = (n - lane + QUEUES - 1) / QUEUES -
                   (long long)__hip_atomic_load(next + lane * QSTRIDE, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t some = __ballot(left > 0), after = some & (~0ull << (qj + 1));
        if (!some) done = true;
        else qj = __ffsll((unsigned long long)(after ? after : some)) - 1;
    }
    return got;
}

// The launch of the skewed band (verify_ring.hip): pairs in the class order of ring_class,
// off[] the bin offsets of that order (bins per class: RING_BINS, widest class first).
using PersistClassKernel = void (*)(const uint64_t *, const int64_t *, const uint32_t *, VSet, VSet,
                                    int, uint8_t *, unsigned long long *, unsigned long long *);
PersistClassKernel ring_kernel(int np, int cmax);  // bands of up to cmax words
// Lanes per half (G) and words per lane (W) of each class; a class holds bands of
// K <= 32 W (G - 2).
constexpr int RING_CLASSES = 6;
constexpr int RING_G[RING_CLASSES] = {4, 8, 16, 16, 16, 16};
constexpr int RING_W[RING_CLASSES] = {1, 1, 1, 2, 3, 5};
constexpr int RING_BINS = 512;  // length bins per class
__host__ __device__ __forceinline__ int ring_class(int32_t K) {
    int c = 0;
    while (c + 1 < RING_CLASSES && 32 * RING_W[c] * (RING_G[c] - 2) < K) c++;
    return c;
}

// The block filter (verify_filter.hip): flags[i] = 0 for the pairs it rejects, 1 for those
// left to verify (n, or *ndev, pairs; ids valid).
constexpr int BF_K_MIN = 64;
constexpr int64_t BF_MIN_PAIRS = 4096;
bool block_filter_applies(int bits, int cmax, int64_t n);
void block_filter(const uint64_t *pairs, int64_t n, const DevStrings &A, const DevStrings &B,
                  int kmode, uint8_t *flags, hipStream_t s, const uint32_t *ndev);

inline VSet vset(const DevStrings &d) {
    return VSet{d.n, d.offsets, d.len, d.kk, d.planes};
}

}  // namespace mj
