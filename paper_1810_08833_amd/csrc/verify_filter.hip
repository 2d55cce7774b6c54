// Block filter of the batched verification: rejects most pairs that are far apart before
// their band is computed.
//
// Cut the shorter string Y into blocks of L symbols.  An alignment of cost <= K leaves all
// but K of the blocks untouched, and an untouched block stands in the longer string X on a
// band diagonal.  So a pair with more than K blocks that do not is beyond K.  (The pigeonhole
// argument of q-gram and partition filters; Navarro's survey of approximate string matching,
// 2001, Sec. 8.)  A wave takes a pair.  It walks both strings in chunks of 64 L symbols:
// each lane enters the L block codes that start at its L symbols of X's chunk into a table in
// LDS, one byte a code holding the number of the chunk that held it last, then looks up its
// one block of Y's chunk.  A block counts as found when the last chunk that held its code
// reaches into the band: chunks after Y's band are not entered yet, so a code whose last
// chunk lies before the band is on none of its diagonals.  (Whole chunks and symbols around X
// only find more blocks, so no pair within K is rejected.)
//
// What bounds it: LDS, busy 0.65 of the time (393 K pairs of 5,500 symbols, 1.29 ms), half of that
// with bank conflicts of the table's byte writes and look-ups at random codes; VALU 0.41, about 60
// instructions per chunk, 9 lane operations a symbol where the band recurrence takes 13 for each of
// its words.  Short strings and pairs within K cost it more than it saves: the verifier times
// whether to run it.  The strings come in
// segments of eight chunks through LDS, 16 bytes a lane, loaded a pair ahead (the first
// segment) or a segment ahead: with each lane loading its own chunk's words one chunk ahead
// the kernel waited on memory nearly all the time (393 K pairs of 5,500 symbols: 5.6 ms).
#include <algorithm>

#include "mj_common.h"
#include "verify_common.h"

namespace mj {

constexpr int BF_L = 7;                // symbols a block: codes of 14 bits, 2 planes
constexpr int BF_C = 64 * BF_L;        // symbols a chunk
constexpr int BF_SEG = 8;              // chunks a segment
constexpr int BF_TABLE = 1 << (2 * BF_L);
constexpr int BF_WORDS = 128;          // plane words one load of 16 bytes a lane brings
// a segment's symbols, a code's length and the alignment of its first word fit one load; so
// do, with a second one, the chunks before it that reach into the first chunk's band
static_assert(BF_SEG * BF_C + 2 * BF_L + 64 <= 32 * BF_WORDS, "segment");
constexpr int BF_BACK_MAX = (2 * 32 * BF_WORDS - BF_SEG * BF_C - 2 * BF_L - 64) / BF_C;

// flags[i] = 0 for the pairs i < n (or *ndev) that are beyond K, 1 for those left to verify:
// all with K < k_min among them (their bands cost less than this).  2 planes, codes below 4.
__global__ __launch_bounds__(64) void k_block_filter(const uint64_t *__restrict__ pairs, int64_t n,
                                                     VSet A, VSet B, int kmode, int k_min,
                                                     uint8_t *__restrict__ flags,
                                                     const uint32_t *__restrict__ ndev) {
    if (ndev) n = min(n, (int64_t)*ndev);
    __shared__ __attribute__((aligned(16))) uint8_t last[BF_TABLE];
    __shared__ __attribute__((aligned(16))) uint2 xs[2 * BF_WORDS + 2], ys[BF_WORDS + 2];
    const int lane = threadIdx.x;
    const int64_t nw = gridDim.x;
    uint32_t stamp0 = 255;  // stamps up to this are older pairs' (255: the table must be cleared)
    for (int64_t b0 = blockIdx.x; b0 < n; b0 += 64 * nw) {
        // a lane loads what is to be known of one of the wave's next 64 pairs
        const int64_t mine = b0 + lane * nw;
        int32_t vK = 0, vmp = 0, vnt = 0;
        int64_t vx = 0, vy = 0;  // global numbers of the strings' first symbols
        bool vxb = false, near = false, test = false;
        if (mine < n) {
            const uint64_t pr = pairs[mine];
            const int32_t ia = (int32_t)(pr >> 32), ib = (int32_t)(uint32_t)pr;
            const int32_t ma = A.len[ia], mb = B.len[ib];
            vK = kmode == 0 ? max(A.kk[ia], B.kk[ib]) : A.kk[ia];
            vxb = ma < mb;
            vmp = max(ma, mb);
            vnt = min(ma, mb);
            vx = vxb ? B.off[ib] : A.off[ia];
            vy = vxb ? A.off[ia] : B.off[ib];
            near = vmp - vnt <= vK;
            const int nb = vnt / BF_L, back = (vK + BF_C - 1) / BF_C, nch = (nb + 63) >> 6;
            test = near && vK >= k_min && nb > vK && back <= BF_BACK_MAX && back + nch <= 254;
        }
        uint64_t keep = __ballot(near && !test);
        uint64_t todo = __ballot(test);
        struct Pair {
            int K, mp, nt, bhi, back, nch;
            int64_t offx, offy, fx, fy;  // first symbols; first staged plane words (even)
            const uint32_t *px, *py;
        };
        auto lane64 = [](int64_t v, int q) -> int64_t {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, q);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), q);
            return (int64_t)(((uint64_t)hi << 32) | lo);
        };
        auto pair_of = [&](int q) {
            Pair r;
            r.K = __builtin_amdgcn_readlane(vK, q);
            r.mp = __builtin_amdgcn_readlane(vmp, q);
            r.nt = __builtin_amdgcn_readlane(vnt, q);
            const int dlen = r.mp - r.nt;
            r.bhi = (r.K + dlen) >> 1;
            // chunks of X that reach into the band of a chunk of Y, besides its own
            r.back = (r.bhi + ((r.K - dlen) >> 1) + BF_C - 1) / BF_C;
            r.nch = (r.nt / BF_L + 63) >> 6;
            r.offx = lane64(vx, q);
            r.offy = lane64(vy, q);
            const bool xb = __builtin_amdgcn_readlane(vxb ? 1 : 0, q) != 0;
            r.px = xb ? B.planes : A.planes;
            r.py = xb ? A.planes : B.planes;
            r.fx = ((r.offx + r.bhi - (int64_t)r.back * BF_C) >> 5) & ~1ll;
            r.fy = (r.offy >> 5) & ~1ll;
            return r;
        };
        // words w0 + 2 lane and the next one of a string's planes, none past its last symbol's
        auto fetch = [&](const uint32_t *planes, int64_t w0, int64_t end) -> uint4 {
            const int64_t wd = w0 + 2 * lane;
            uint4 v = {0u, 0u, 0u, 0u};
            if (wd >= 0 && wd <= end >> 5) v = *reinterpret_cast<const uint4 *>(planes + 2 * wd);
            return v;
        };
        uint4 x0, x1, y0, xn, yn;
        if (todo) {
            const Pair r = pair_of(__ffsll((unsigned long long)todo) - 1);
            x0 = fetch(r.px, r.fx, r.offx + r.mp);
            x1 = fetch(r.px, r.fx + BF_WORDS, r.offx + r.mp);
            y0 = fetch(r.py, r.fy, r.offy + r.nt);
        }
        while (todo) {
            const int q = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const Pair r = pair_of(q);
            const int nblocks = r.nt / BF_L;
            reinterpret_cast<uint4 *>(xs)[lane] = x0;
            reinterpret_cast<uint4 *>(xs)[64 + lane] = x1;
            reinterpret_cast<uint4 *>(ys)[lane] = y0;
            if (todo) {  // the next pair's first segment
                const Pair t = pair_of(__ffsll((unsigned long long)todo) - 1);
                x0 = fetch(t.px, t.fx, t.offx + t.mp);
                x1 = fetch(t.px, t.fx + BF_WORDS, t.offx + t.mp);
                y0 = fetch(t.py, t.fy, t.offy + t.nt);
            }
            if (stamp0 + (uint32_t)(r.back + r.nch) > 255u) {
                const uint4 z = {0u, 0u, 0u, 0u};
                for (int j = lane; j < BF_TABLE / 16; j += 64) reinterpret_cast<uint4 *>(last)[j] = z;
                stamp0 = 0;
            }
            int missed = 0;
            bool far = false, over = false;
            int m = -r.back;  // X's next chunk: symbols r.bhi + C m .., stamp stamp0 + 1 + back + m
            for (int k0 = 0; k0 < r.nch && !over; k0 += BF_SEG) {
                // the staged words' first symbols, relative to X's and Y's
                int bx = (int)(r.fx * 32 - r.offx), by = (int)(r.fy * 32 - r.offy);
                if (k0 > 0) {
                    const int64_t wx = ((r.offx + r.bhi + (int64_t)BF_C * k0) >> 5) & ~1ll;
                    const int64_t wy = ((r.offy + (int64_t)BF_C * k0) >> 5) & ~1ll;
                    bx = (int)(wx * 32 - r.offx);
                    by = (int)(wy * 32 - r.offy);
                    reinterpret_cast<uint4 *>(xs)[lane] = xn;
                    reinterpret_cast<uint4 *>(ys)[lane] = yn;
                }
                if (k0 + BF_SEG < r.nch) {  // the next segment
                    const int64_t kn = (int64_t)BF_C * (k0 + BF_SEG);
                    xn = fetch(r.px, ((r.offx + r.bhi + kn) >> 5) & ~1ll, r.offx + r.mp);
                    yn = fetch(r.py, ((r.offy + kn) >> 5) & ~1ll, r.offy + r.nt);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                // this lane's symbols: X's from r.bhi + C m + L lane on, Y's from C k + L lane
                const int rx = r.bhi + BF_L * lane - bx, ry = BF_L * lane - by;
                auto window = [](const uint2 *st, int at, uint32_t &w0, uint32_t &w1) {
                    const uint2 lo = st[at >> 5], hi = st[(at >> 5) + 1];
                    w0 = __builtin_amdgcn_alignbit(hi.x, lo.x, (uint32_t)at & 31u);
                    w1 = __builtin_amdgcn_alignbit(hi.y, lo.y, (uint32_t)at & 31u);
                };
                auto code = [](uint32_t w0, uint32_t w1, int t) -> uint32_t {
                    return __builtin_amdgcn_ubfe(w0, (unsigned)t, (unsigned)BF_L) |
                           (__builtin_amdgcn_ubfe(w1, (unsigned)t, (unsigned)BF_L) << BF_L);
                };
                uint32_t xa, xb, ya, yb, na, nb, ma, mb;
                window(xs, rx + BF_C * m, xa, xb);
                window(ys, ry + BF_C * k0, ya, yb);
                const int kend = min(k0 + BF_SEG, r.nch);
                for (int k = k0; k < kend;) {
                    // the next chunk's windows while this one's codes are entered
                    window(xs, rx + BF_C * (m + 1), na, nb);
                    const uint8_t st = (uint8_t)(stamp0 + 1u + (uint32_t)(r.back + m));
#pragma unroll
                    for (int t = 0; t < BF_L; t++) last[code(xa, xb, t)] = st;
                    xa = na;
                    xb = nb;
                    if (m++ < k) continue;
                    window(ys, ry + BF_C * (k + 1), ma, mb);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    const bool miss = (uint32_t)last[code(ya, yb, 0)] < stamp0 + 1u + (uint32_t)k &&
                                      64 * k + lane < nblocks;
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    missed += (int)__popcll(__ballot(miss));
                    k++;
                    far = missed > r.K;
                    over = far || missed + (nblocks - 64 * k) <= r.K;  // rejected, or never to be
                    if (over) break;
                    ya = ma;
                    yb = mb;
                }
            }
            stamp0 += (uint32_t)(r.back + r.nch);
            if (!far) keep |= 1ull << q;
        }
        if (mine < n) flags[mine] = (uint8_t)((keep >> lane) & 1u);
    }
}

bool block_filter_applies(int bits, int cmax, int64_t n) {
    return bits == 2 && 32 * cmax >= BF_K_MIN && n >= BF_MIN_PAIRS;
}

void block_filter(const uint64_t *pairs, int64_t n, const DevStrings &A, const DevStrings &B,
                  int kmode, uint8_t *flags, hipStream_t s, const uint32_t *ndev) {
    if (n <= 0) return;
    // eight waves of a CU hold their tables and segments (19 of 160 KB each)
    const unsigned grid = (unsigned)std::min<int64_t>(n, 256 * 8);
    hipLaunchKernelGGL(k_block_filter, dim3(grid), dim3(64), 0, s, pairs, n, vset(A), vset(B), kmode,
                       BF_K_MIN, flags, ndev);
    MJ_LAUNCH_CHECK();
}

}  // namespace mj
