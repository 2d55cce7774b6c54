// Grouping, pair tests and dedup in LDS: radix passes by the top key bits bring the records
// of a group together (buckets of about BK_AVG records), and a workgroup takes a bucket at a
// time.
//
//   k_bucket_pairs  finds a bucket's members (records whose key may occur twice) with two LDS
//                   bitmaps over 15 more key bits and brings those alone together by slots of
//                   11 of them, so that the records of a group (equal keys, Alg. 3's hash table
//                   D) share a slot; every member is tested against half of its slot, cyclically.
//                   No record is sorted by its full key, no group bounded, no pair test numbered.
//                   Beyond 2^23 records the same goes over the member filter's records.
//   k_long_pairs    slots of more than BK_LONG records (frequent keys), set aside by the first
//                   kernel: a wave per 64 x 64 tile of their pairs.
//   k_dedup_buckets the candidates after one or two radix passes by their top bits, each
//                   bucket sorted in LDS and its distinct pairs kept; k_dedup_gather packs
//                   the buckets' results together.
//
// What bounds a small join is its launches, about 5 us each: these take about 13 where the
// record sort with its repair, the group stage, the emission and the dedup took 48.  A join
// whose buckets do not fit their LDS is seen by its counts and goes by the general path.
#include <algorithm>

#include "bucket_plan.h"
#include "mj_common.h"

namespace mj {

constexpr int BK_THREADS = 512, BK_WAVES = BK_THREADS / 64;
constexpr int BK_MTHREADS = 256;  // of a workgroup where all records are members
constexpr int BK_KEEP = 4, BK_MKEEP = 2;  // of a bucket's records each thread keeps in registers
constexpr int BK_SUB = 15;      // key bits of a bucket's bitmaps; log2 BK_SLOTS of them number the slot
constexpr int BK_SLOTS = 2048, BK_MSLOTS = 1024;
constexpr int BK_STAGE = 512;   // candidates staged before they take room in the output
constexpr int BK_LONG = 63;     // slots of more records are set aside
constexpr int BK_CHUNK = 64;    // buckets whose bounds are found together
constexpr int BK_LONGS = 64;    // such slots of a bucket
constexpr int BK_DISTINCT = 32; // distinct keys of such a slot
static_assert(2 * DD_CAP == 1 << DD_LOG, "dedup table");

// First index in [0, n) whose key's top bits are >= b, by the whole wave: a 64-way search.
__device__ __forceinline__ int64_t bucket_start(const uint64_t *__restrict__ key, int64_t n,
                                                int shift, uint64_t b) {
    const int lane = threadIdx.x & 63;
    int64_t lo = 0, hi = n;  // the answer is in [lo, hi]
    while (hi > lo) {
        const int64_t step = (hi - lo + 63) / 64;
        const int64_t at = lo + (int64_t)(lane + 1) * step - 1;  // last of the lane's part
        const bool below = at < hi && (key[at] >> shift) < b;
        const int c = __popcll(__ballot(below));  // parts wholly below
        const int64_t nlo = min(hi, lo + (int64_t)c * step);
        hi = min(hi, nlo + step - 1);
        lo = nlo;
    }
    return lo;
}

// A slot's word: the place of its next member (bits 0 .. 15), its size or, of a long slot, its
// number among them (16 .. 29), and whether it is a long one or has fewer than two members.
constexpr uint32_t SLOT_LONG = 1u << 31, SLOT_LONE = 1u << 30;
template <bool MEMBERS>
struct BucketShared {
    static constexpr int THREADS = MEMBERS ? BK_MTHREADS : BK_THREADS, WAVES = THREADS / 64;
    static constexpr int SLOTS = MEMBERS ? BK_MSLOTS : BK_SLOTS;
    uint64_t key[BK_CAP];    // members by slot
    int4 rec[BK_CAP];        // their string id, m, 2 pos - m, K
    uint64_t stage[BK_STAGE];
    uint32_t seen[MEMBERS ? 4 : 1 << (BK_SUB - 5)], again[MEMBERS ? 4 : 1 << (BK_SUB - 5)];
    uint32_t slot[SLOTS];
    uint32_t bin[64];        // short slots' members by the size of their slots, then their places
    uint32_t lcount[BK_LONGS], lfill[BK_LONGS];  // long slots: records, those placed
    int64_t lbase[BK_LONGS];
    uint32_t nlong, nstage, members;
    unsigned long long sbase;
    uint64_t found[BK_DISTINCT];
    uint32_t least, same;
    int64_t bound[BK_CHUNK + 2];
};

// What the kernels read and write.  Records are grouped by their keys' top `bits` bits; n from
// *n_dev when given.
struct BucketIn {
    const uint64_t *key, *val;
    int64_t n;
    const int64_t *n_dev;
    int bits;
    const int32_t *len, *kk;
};
struct BucketOut {
    uint64_t *out;  // candidates, cap of them; their number (which may be more) to *counter
    int64_t cap;
    unsigned long long *counter;
    uint64_t *part;  // by workgroup: pair tests, groups of two or more, members
    uint32_t *over;  // set when a bucket does not fit
    // records of the long slots, and (first, count) of each slot; *xstate = slots << 40 | records
    uint64_t *xkey;
    int4 *xrec;
    int64_t xcap;
    ulonglong2 *xslot;
    int64_t xslots;
    unsigned long long *xstate;
    uint64_t max_units;  // tile pairs of the long slots that are taken on
};

// For inputs of fewer than 2^29 symbols (32-bit filter).  MEMBERS: the records are those the
// member filter kept, so no bitmaps are needed.
//
// A bucket is a chain of short steps between barriers, so what bounds the kernel is how many
// workgroups a CU holds and what each step waits for: the next bucket's records and this one's
// lengths are loaded ahead (MEMBERS: 256 threads; a CU's registers hold four such workgroups, or
// two of 512 threads, and the grid is that many: half a round more, six a CU, left the device half
// empty at the end), the bounds of 64 buckets found at once, and short slots laid out by size, so that a wave's lanes have about
// as many tests each.  Room in the output is taken in pieces of 256 candidates or more, since
// one address takes 80 M atomics a second; a bucket of more than the stage holds is tested twice.
// 17.3 M members, 256 M tests, 10.1 M candidates: 0.98 ms with the long slots' 0.27, with as many
// workgroups as fit at once 0.86, where the two more sort passes, the repair, the groups and the
// emission took 1.9 ms; with a wave's candidates straight to the output and slots in key order
// 1.74 ms.  7.0 M unfiltered records (0.41 M groups): 167 us with twice the workgroups that fit,
// 159 with those.
template <bool MEMBERS>
__global__ __launch_bounds__(MEMBERS ? BK_MTHREADS : BK_THREADS) void k_bucket_pairs(BucketIn in,
                                                                                    BucketOut o) {
    using Shared = BucketShared<MEMBERS>;
    constexpr int BK_THREADS = Shared::THREADS, BK_WAVES = Shared::WAVES, BK_SLOTS = Shared::SLOTS;
    constexpr int BK_KEEP = MEMBERS ? BK_MKEEP : mj::BK_KEEP;
    __shared__ __attribute__((aligned(16))) Shared sh;
    const int64_t n = in.n_dev ? min(in.n, *in.n_dev) : in.n;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, bits = in.bits;
    const int64_t nb = 1ll << bits;
    const int64_t b0 = nb * blockIdx.x / gridDim.x, b1 = nb * (blockIdx.x + 1) / gridDim.x;
    uint64_t tests = 0, groups = 0, members = 0;  // this thread's
    if (threadIdx.x == 0) sh.nstage = 0;
    // passing pairs (whole wave; up to two a lane, of string a) into the stage, counted beyond
    // its room; `out` >= 0: to there
    auto emit = [&](bool p0, bool p1, int a, int c0, int c1, int64_t out) {
        const uint64_t m0 = __ballot(p0), m1 = __ballot(p1), low = (1ull << lane) - 1;
        if (!(m0 | m1)) return;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&sh.nstage, (uint32_t)(__popcll(m0) + __popcll(m1)));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        auto put = [&](uint32_t i, int c) {
            const uint64_t pr = ((uint64_t)(uint32_t)min(a, c) << 32) | (uint32_t)max(a, c);
            if (out >= 0) {
                if (out + i < o.cap) o.out[out + i] = pr;
            } else if (i < BK_STAGE) {
                sh.stage[i] = pr;
            }
        };
        if (p0) put(at + (uint32_t)__popcll(m0 & low), c0);
        if (p1) put(at + (uint32_t)(__popcll(m0) + __popcll(m1 & low)), c1);
    };
    auto flush = [&](bool all) {  // whole workgroup, after a barrier
        const uint32_t staged = sh.nstage;
        if (staged == 0 || (!all && staged < BK_STAGE / 2)) return;
        if (threadIdx.x == 0) sh.sbase = atomicAdd(o.counter, (unsigned long long)staged);
        __syncthreads();
        const unsigned long long g = sh.sbase;
        for (uint32_t i = threadIdx.x; i < staged; i += BK_THREADS)
            if ((int64_t)(g + i) < o.cap) o.out[g + i] = sh.stage[i];
        __syncthreads();
        if (threadIdx.x == 0) sh.nstage = 0;
        __syncthreads();
    };
    // BK_SUB key bits besides the bucket's (records of equal key agree on them)
    auto sub = [](uint64_t e) -> uint32_t { return (uint32_t)e & ((1u << BK_SUB) - 1); };
    for (int64_t c0 = b0; c0 < b1; c0 += BK_CHUNK) {
        // the bounds of the next buckets: the outer two a wave each, those between a wave each
        // where they are few (three steps of a 64-way search), else a thread each
        const int nc = (int)min((int64_t)BK_CHUNK, b1 - c0);
        __syncthreads();
        if (wv < 2) {
            const int64_t b = c0 + (wv ? nc : 0);
            const int64_t at = b == 0 ? 0 : b == nb ? n : bucket_start(in.key, n, 64 - bits, (uint64_t)b);
            if (lane == 0) sh.bound[wv ? nc : 0] = at;
        }
        __syncthreads();
        if (nc <= BK_WAVES + 1) {
            const int64_t a = sh.bound[0], z = sh.bound[nc];
            if (wv + 1 < nc) {
                const int64_t at = a + bucket_start(in.key + a, z - a, 64 - bits, (uint64_t)(c0 + wv + 1));
                if (lane == 0) sh.bound[wv + 1] = at;
            }
        }
        for (int i = 1 + (int)threadIdx.x; i < nc && nc > BK_WAVES + 1; i += BK_THREADS) {
            int64_t a = sh.bound[0], z = sh.bound[nc];
            while (a < z) {
                const int64_t mid = (a + z) >> 1;
                if (in.key[mid] >> (64 - bits) < (uint64_t)(c0 + i)) a = mid + 1;
                else z = mid;
            }
            sh.bound[i] = a;
        }
        if (threadIdx.x == 0) sh.bound[nc + 1] = sh.bound[nc];  // (an empty one after the last)
        __syncthreads();
        // MEMBERS: a bucket's records are loaded while the one before it is worked on
        uint64_t nx[BK_KEEP], nv[BK_KEEP];
        auto load = [&](int64_t lo, int64_t m, uint64_t *x, uint64_t *v) {
#pragma unroll
            for (int u = 0; u < BK_KEEP; u++) {
                const int64_t i = threadIdx.x + u * BK_THREADS;
                x[u] = i < m ? in.key[lo + i] : 0;
                if (MEMBERS) v[u] = i < m ? in.val[lo + i] : 0;
            }
        };
        if (MEMBERS) load(sh.bound[0], sh.bound[1] - sh.bound[0], nx, nv);
        for (int c = 0; c < nc; c++) {
            const int64_t lo = sh.bound[c], m = sh.bound[c + 1] - lo;
            const bool keep = m <= BK_KEEP * BK_THREADS;
            uint64_t x[BK_KEEP], v[BK_KEEP];
            if (MEMBERS) {
#pragma unroll
                for (int u = 0; u < BK_KEEP; u++) {
                    x[u] = nx[u];
                    v[u] = nv[u];
                }
                load(sh.bound[c + 1], sh.bound[c + 2] - sh.bound[c + 1], nx, nv);
            } else if (keep) {
                load(lo, m, x, v);
            }
            if (m < 2) continue;  // (uniform)
            int32_t ml[BK_KEEP], ks[BK_KEEP];
            auto strings = [&](int u, bool need) {
                ml[u] = need ? in.len[v[u] >> 32] : 0;
                ks[u] = need ? in.kk[v[u] >> 32] : 0;
            };
            if (MEMBERS)
#pragma unroll
                for (int u = 0; u < BK_KEEP; u++) strings(u, threadIdx.x + u * BK_THREADS < m);
            auto each = [&](auto f) {
                if (keep) {
#pragma unroll
                    for (int u = 0; u < BK_KEEP; u++)
                        if (threadIdx.x + u * BK_THREADS < m) f(x[u], (int64_t)threadIdx.x + u * BK_THREADS);
                } else {
                    for (int64_t i = threadIdx.x; i < m; i += BK_THREADS) f(in.key[lo + i], i);
                }
            };
            {
                const uint4 z = make_uint4(0u, 0u, 0u, 0u);
                if (!MEMBERS)
                    for (int i = threadIdx.x; i < (1 << (BK_SUB - 7)); i += BK_THREADS) {
                        reinterpret_cast<uint4 *>(sh.seen)[i] = z;
                        reinterpret_cast<uint4 *>(sh.again)[i] = z;
                    }
                for (int i = threadIdx.x; i < BK_SLOTS / 4; i += BK_THREADS)
                    reinterpret_cast<uint4 *>(sh.slot)[i] = z;
                if (threadIdx.x < BK_LONGS) sh.lfill[threadIdx.x] = 0;
                if (threadIdx.x < 64) sh.bin[threadIdx.x] = 0;
                if (threadIdx.x == 0) sh.nlong = 0;
            }
            __syncthreads();
            if (!MEMBERS) {
                each([&](uint64_t e, int64_t) {
                    const uint32_t h = sub(e), bit = 1u << (h & 31);
                    if (atomicOr(&sh.seen[h >> 5], bit) & bit) atomicOr(&sh.again[h >> 5], bit);
                });
                __syncthreads();
            }
            auto member = [&](uint32_t h) { return MEMBERS || ((sh.again[h >> 5] >> (h & 31)) & 1u) != 0; };
            each([&](uint64_t e, int64_t) {
                const uint32_t h = sub(e);
                if (member(h)) atomicAdd(&sh.slot[h & (BK_SLOTS - 1)], 1u);
            });
            __syncthreads();
            // slots to places, those of one size together, the largest first: a thread's
            // BK_SLOTS / BK_THREADS consecutive slots
            {
                constexpr int PER = BK_SLOTS / BK_THREADS;
                uint32_t v[PER];
#pragma unroll
                for (int k = 0; k < PER; k++) {
                    v[k] = sh.slot[threadIdx.x * PER + k];
                    if (v[k] >= 2 && v[k] <= BK_LONG) atomicAdd(&sh.bin[BK_LONG - v[k]], v[k]);
                }
                __syncthreads();
                if (wv == 0) {
                    const uint32_t mine = sh.bin[lane];
                    uint32_t inc = mine;
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const uint32_t y = (uint32_t)__shfl_up((int)inc, d, 64);
                        if (lane >= d) inc += y;
                    }
                    sh.bin[lane] = inc - mine;
                    if (lane == 63) sh.members = inc;
                }
                __syncthreads();
#pragma unroll
                for (int k = 0; k < PER; k++) {
                    uint32_t word = SLOT_LONE;
                    if (v[k] > BK_LONG) {
                        const uint32_t l = atomicAdd(&sh.nlong, 1u);
                        if (l < BK_LONGS) sh.lcount[l] = v[k];
                        word = SLOT_LONG | (min(l, (uint32_t)BK_LONGS - 1) << 16);
                    } else if (v[k] >= 2) {
                        word = min(atomicAdd(&sh.bin[BK_LONG - v[k]], v[k]), 0xFFFFu) | (v[k] << 16);
                    }
                    sh.slot[threadIdx.x * PER + k] = word;
                }
            }
            __syncthreads();
            const uint32_t M = sh.members, nl = sh.nlong;
            if (M > BK_CAP || nl > BK_LONGS) {
                if (threadIdx.x == 0) *o.over = M > BK_CAP ? OVER_MEMBERS : OVER_SLOTS;
                __syncthreads();
                continue;
            }
            if (nl && wv == 0) {  // room for the long slots' records
                const uint32_t cnt = lane < (int)nl ? sh.lcount[lane] : 0u;
                uint32_t inc = cnt;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const uint32_t y = (uint32_t)__shfl_up((int)inc, d, 64);
                    if (lane >= d) inc += y;
                }
                unsigned long long at = 0;
                if (lane == 63) at = atomicAdd(o.xstate, ((unsigned long long)nl << 40) | inc);
                at = (unsigned long long)__shfl((long long)at, 63, 64);
                const int64_t first = (int64_t)(at & ((1ull << 40) - 1)) + (inc - cnt);
                const int64_t d = (int64_t)(at >> 40) + lane;
                const bool room = first + cnt <= o.xcap && d < o.xslots && cnt < (1u << 24);
                if (lane < (int)nl) {
                    if (room) o.xslot[d] = make_ulonglong2((unsigned long long)first, cnt);
                    else *o.over = OVER_ROOM;
                    sh.lbase[lane] = room ? first : -1;
                }
            }
            if (nl) __syncthreads();
            // each member's place: among the short slots' (>= 0), or in its long slot
            // (-1 - (slot << 24 | place)); NONE: no member, or no room
            constexpr int NONE = 1 << 30;
            auto place = [&](uint64_t e) -> int {
                const uint32_t h = sub(e);
                if (!member(h)) return NONE;
                members++;
                const uint32_t wd = sh.slot[h & (BK_SLOTS - 1)];
                if (wd & SLOT_LONE) return NONE;
                if (!(wd & SLOT_LONG)) return (int)(atomicAdd(&sh.slot[h & (BK_SLOTS - 1)], 1u) & 0xFFFFu);
                const uint32_t l = (wd >> 16) & (BK_LONGS - 1);
                if (sh.lbase[l] < 0) return NONE;
                return -1 - (int)((l << 24) | atomicAdd(&sh.lfill[l], 1u));
            };
            auto put = [&](int p, uint64_t k, uint64_t v, int32_t ml, int32_t ks) {
                const int4 rc = make_int4((int32_t)(v >> 32), ml, 2 * (int32_t)(uint32_t)v - ml, ks);
                if (p >= 0) {
                    sh.key[p] = k;
                    sh.rec[p] = rc;
                } else {
                    const uint32_t q = (uint32_t)(-1 - p);
                    const int64_t lp = sh.lbase[q >> 24] + (q & 0xFFFFFFu);
                    o.xkey[lp] = k;
                    o.xrec[lp] = rc;
                }
            };
            if (keep) {  // the loads of a thread's members in flight together
                int p[BK_KEEP];
#pragma unroll
                for (int u = 0; u < BK_KEEP; u++)
                    p[u] = threadIdx.x + u * BK_THREADS < m ? place(x[u]) : NONE;
                if (!MEMBERS) {
#pragma unroll
                    for (int u = 0; u < BK_KEEP; u++)
                        v[u] = p[u] != NONE ? in.val[lo + threadIdx.x + u * BK_THREADS] : 0;
#pragma unroll
                    for (int u = 0; u < BK_KEEP; u++) strings(u, p[u] != NONE);
                }
#pragma unroll
                for (int u = 0; u < BK_KEEP; u++)
                    if (p[u] != NONE) put(p[u], x[u], v[u], ml[u], ks[u]);
            } else {
                for (int64_t i = threadIdx.x; i < m; i += BK_THREADS) {
                    const uint64_t e = in.key[lo + i];
                    const int p = place(e);
                    if (p == NONE) continue;
                    const uint64_t v = in.val[lo + i];
                    put(p, e, v, in.len[v >> 32], in.kk[v >> 32]);
                }
            }
            const uint32_t before = sh.nstage;
            __syncthreads();
            // Members of short slots, one a lane, each against the half of its slot that follows
            // it (cyclically): lanes of one slot have the same number of tests, and neighbouring
            // slots are of one size.
            auto pairs = [&](int64_t out) {
                for (int p0 = 64 * wv; p0 < (int)M; p0 += BK_THREADS) {
                    const int p = p0 + lane;
                    int first = 0, z = 0, nd = 0;
                    uint64_t kp = 0;
                    int4 u = {};
                    if (p < (int)M) {
                        kp = sh.key[p];
                        u = sh.rec[p];
                        const uint32_t wd = sh.slot[(uint32_t)kp & (BK_SLOTS - 1)];
                        z = (int)(wd >> 16);
                        first = (int)(wd & 0xFFFFu) - z;
                        nd = (z - 1) / 2 + (z % 2 == 0 && p - first < z / 2 ? 1 : 0);
                        if (out < 0) {  // a group's first member in the slot, with another after it
                            int q = p - 1;
                            while (q >= first && sh.key[q] != kp) q--;
                            if (q < first) {
                                q = p + 1;
                                while (q < first + z && sh.key[q] != kp) q++;
                                groups += q < first + z ? 1 : 0;
                            }
                        }
                    }
                    uint32_t same = 0;
                    int q = p;
                    auto close = [&](const int4 &v) {
                        return u.x != v.x && (uint32_t)max(abs(u.y - v.y), abs(u.z - v.z)) <=
                                                 max((uint32_t)u.w, (uint32_t)v.w);
                    };
                    for (int d = 1; __any(d <= nd); d += 2) {
                        const int q0 = q + 1 >= first + z ? first : q + 1;
                        q = q0 + 1 >= first + z ? first : q0 + 1;
                        const bool e0 = d <= nd && sh.key[q0] == kp, e1 = d < nd && sh.key[q] == kp;
                        same += (e0 ? 1u : 0u) + (e1 ? 1u : 0u);
                        const int4 v0 = sh.rec[e0 ? q0 : 0], v1 = sh.rec[e1 ? q : 0];
                        emit(e0 && close(v0), e1 && close(v1), u.x, v0.x, v1.x, out);
                    }
                    if (out < 0) tests += same;
                }
            };
            pairs(-1);
            __syncthreads();
            const uint32_t staged = sh.nstage;
            if (staged > BK_STAGE) {  // this bucket's straight to the output, in one piece
                __syncthreads();
                if (threadIdx.x == 0) {
                    sh.sbase = atomicAdd(o.counter, (unsigned long long)(staged - before));
                    sh.nstage = 0;
                }
                __syncthreads();
                pairs((int64_t)sh.sbase);
                __syncthreads();
                if (threadIdx.x == 0) sh.nstage = before;
            }
            // long slots: how often each of their (few) distinct keys occurs
            for (uint32_t l = 0; l < nl; l++) {
                const int64_t first = sh.lbase[l];
                const uint32_t cnt = sh.lcount[l];
                if (first < 0) continue;
                uint32_t left = cnt;
                for (int k = 0; left > 0; k++) {
                    if (k == BK_DISTINCT) {
                        if (threadIdx.x == 0) *o.over = OVER_DISTINCT;
                        break;
                    }
                    if (threadIdx.x == 0) {
                        sh.least = k ? ~0u : 0u;
                        sh.same = 0;
                    }
                    __syncthreads();
                    uint32_t least = k ? ~0u : 0u;  // the first record whose key is not among the k found
                    for (uint32_t i = threadIdx.x; i < cnt && least == ~0u; i += BK_THREADS) {
                        const uint64_t y = o.xkey[first + i];
                        bool known = false;
                        for (int j = 0; j < k; j++) known = known || sh.found[j] == y;
                        if (!known) least = i;
                    }
                    if (k && least != ~0u) atomicMin(&sh.least, least);
                    __syncthreads();
                    const uint64_t y = o.xkey[first + sh.least];
                    uint32_t mine = 0;
                    for (uint32_t i = threadIdx.x; i < cnt; i += BK_THREADS) mine += o.xkey[first + i] == y;
                    if (mine) atomicAdd(&sh.same, mine);
                    if (threadIdx.x == 0) sh.found[k] = y;
                    __syncthreads();
                    const uint32_t z = sh.same;
                    left -= z;
                    if (threadIdx.x == 0) {
                        tests += (uint64_t)z * (z - 1) / 2;
                        groups += z >= 2 ? 1 : 0;
                    }
                    __syncthreads();
                }
            }
            __syncthreads();
            flush(false);
        }
    }
    __syncthreads();
    flush(true);
    // this workgroup's sums
    for (int d = 32; d >= 1; d >>= 1) {
        tests += (uint64_t)__shfl_down((long long)tests, d, 64);
        groups += (uint64_t)__shfl_down((long long)groups, d, 64);
        members += (uint64_t)__shfl_down((long long)members, d, 64);
    }
    __syncthreads();
    if (lane == 0) {
        sh.stage[3 * wv] = tests;
        sh.stage[3 * wv + 1] = groups;
        sh.stage[3 * wv + 2] = members;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint64_t t = 0;
        for (int w = 0; w < BK_WAVES; w++) t += sh.stage[3 * w + threadIdx.x];
        o.part[3 * blockIdx.x + threadIdx.x] = t;
    }
}

// ustart[d] = the 64 x 64 tile pairs of the long slots before slot d; ustart[slots] = all.
constexpr int LU_ITEMS = 8;
__global__ __launch_bounds__(BK_THREADS) void k_long_units(const ulonglong2 *__restrict__ xslot,
                                                           int64_t xslots,
                                                           const unsigned long long *xstate,
                                                           uint64_t *__restrict__ ustart) {
    __shared__ uint64_t tmp[BK_WAVES];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t d = min(xslots, (int64_t)(*xstate >> 40));
    uint64_t run = 0;  // the units of the slots before this chunk
    for (int64_t c0 = 0; c0 < d; c0 += BK_THREADS * LU_ITEMS) {
        const int64_t i0 = c0 + (int64_t)threadIdx.x * LU_ITEMS;
        uint64_t v[LU_ITEMS], sum = 0;
#pragma unroll
        for (int k = 0; k < LU_ITEMS; k++) v[k] = i0 + k < d ? xslot[i0 + k].y : 0;
#pragma unroll
        for (int k = 0; k < LU_ITEMS; k++) {
            const uint64_t nt = (v[k] + 63) / 64;
            v[k] = sum;
            sum += nt * (nt + 1) / 2;
        }
        uint64_t inc = sum;
        for (int s = 1; s < 64; s <<= 1) {
            const uint64_t y = (uint64_t)__shfl_up((long long)inc, s, 64);
            if (lane >= s) inc += y;
        }
        __syncthreads();
        if (lane == 63) tmp[wv] = inc;
        __syncthreads();
        uint64_t at = run + inc - sum;
        for (int w = 0; w < BK_WAVES; w++) {
            if (w < wv) at += tmp[w];
            run += tmp[w];
        }
#pragma unroll
        for (int k = 0; k < LU_ITEMS; k++)
            if (i0 + k < d) ustart[i0 + k] = at + v[k];
    }
    if (threadIdx.x == 0) ustart[d] = run;
}

// A wave takes a share of the tile pairs I <= J in order: lane l holds record 64 I + l, tile
// J's records are read from LDS by all lanes at once.  Candidates are staged by the wave, up to
// LP_BUF of them, since what bounds the kernel where most pairs pass is the one counter (80 M
// atomics a second); a tile pair whose first rows are full finds all its candidates first and
// takes their room at once.  59 M candidates of 4 groups of 1,500: 0.80 -> 0.34 ms with the
// short slots' kernel, 21 M of 20 groups of 400: 0.35 -> 0.20; taking room so at every tile pair
// was 0.29 and 0.17 there, but 0.09 ms more on 17 M members of protein-like strings (0.87), whose
// tile pairs are mostly thin.
constexpr int LP_WAVES = 4, LP_BUF = 1024;
constexpr int LP_LOOK = 4, LP_DENSE = 64;  // rows looked at, candidates of theirs
__global__ __launch_bounds__(64 * LP_WAVES) void k_long_pairs(const uint64_t *__restrict__ ustart,
                                                              BucketOut o) {
    __shared__ uint64_t tkey[LP_WAVES][64];
    __shared__ int4 trec[LP_WAVES][64];
    __shared__ uint64_t buf[LP_WAVES][LP_BUF];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t slots = min(o.xslots, (int64_t)(*o.xstate >> 40));
    if (slots == 0 || *o.over) return;
    const uint64_t units = ustart[slots];
    if (units > o.max_units) {  // more than a pass of tests: the general path counts them first
        if (blockIdx.x == 0 && threadIdx.x == 0) *o.over = OVER_UNITS;
        return;
    }
    const uint64_t waves = (uint64_t)gridDim.x * LP_WAVES, w = (uint64_t)blockIdx.x * LP_WAVES + wv;
    uint64_t u = units * w / waves;
    const uint64_t uend = units * (w + 1) / waves;
    if (u >= uend) return;
    // the slot of the first unit: the last d with ustart[d] <= u
    int64_t d = 0;
    for (int64_t hi = slots; hi - d > 1;) {
        const int64_t step = (hi - d + 63) / 64, at = d + (int64_t)lane * step;
        const int c = __popcll(__ballot(at < hi && ustart[at] <= u));  // lane 0 always
        const int64_t nd = d + (int64_t)(c - 1) * step;
        hi = min(hi, nd + step);
        d = nd;
    }
    uint32_t staged = 0;  // (wave-uniform)
    uint64_t *wb = buf[wv];
    auto drain = [&]() {
        unsigned long long g = 0;
        if (lane == 0) g = atomicAdd(o.counter, (unsigned long long)staged);
        g = (unsigned long long)__shfl((long long)g, 0, 64);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (uint32_t i = lane; i < staged; i += 64)
            if ((int64_t)(g + i) < o.cap) o.out[g + i] = wb[i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        staged = 0;
    };
    const uint64_t in = u - ustart[d];
    uint64_t J = (uint64_t)((sqrt(8.0 * (double)in + 1.0) - 1.0) * 0.5);
    while (J > 0 && J * (J + 1) / 2 > in) J--;
    while ((J + 1) * (J + 2) / 2 <= in) J++;
    uint64_t I = in - J * (J + 1) / 2;
    ulonglong2 sl = o.xslot[d];
    int64_t loaded = -1;
    for (;;) {
        const int64_t z = (int64_t)sl.y, ra = (int64_t)I * 64 + lane;
        const bool ha = ra < z;
        uint64_t ka = 0;
        int4 xa = {};
        if (ha) {
            ka = o.xkey[sl.x + ra];
            xa = o.xrec[sl.x + ra];
        }
        if ((int64_t)J != loaded) {
            const int64_t rb = (int64_t)J * 64 + lane;
            uint64_t kb = 0;
            int4 xb = {};
            if (rb < z) {
                kb = o.xkey[sl.x + rb];
                xb = o.xrec[sl.x + rb];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            tkey[wv][lane] = kb;
            trec[wv][lane] = xb;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            loaded = (int64_t)J;
        }
        const int nbx = (int)min<int64_t>(64, z - (int64_t)J * 64);
        const bool diag = I == J;
        auto passes = [&](int j) -> bool {
            const int4 e = trec[wv][j];
            return ha && (!diag || lane < j) && ka == tkey[wv][j] && xa.x != e.x &&
                   (uint32_t)max(abs(xa.y - e.y), abs(xa.z - e.z)) <= max((uint32_t)xa.w, (uint32_t)e.w);
        };
        auto pair = [&](int j) -> uint64_t {
            const int ex = trec[wv][j].x;
            return ((uint64_t)(uint32_t)min(xa.x, ex) << 32) | (uint32_t)max(xa.x, ex);
        };
        uint32_t found = 0;  // (wave-uniform)
        int top = nbx;       // rows from the last on: of the diagonal's the fullest first
        auto stage = [&](int j) {
            const bool pass = passes(j);
            const uint64_t m = __ballot(pass);
            if (m) {
                if (pass) wb[staged + __popcll(m & ((1ull << lane) - 1))] = pair(j);
                staged += (uint32_t)__popcll(m);
                found += (uint32_t)__popcll(m);
                if (staged > LP_BUF - 64) drain();
            }
        };
        for (int r = 0; r < LP_LOOK && top > 0; r++) stage(--top);
        if (found < LP_DENSE) {
            while (top > 0) stage(--top);
        } else if (top > 0) {
            uint64_t row = 0;  // lane j: the records of tile I that pass with record j of tile J
            for (int j = 0; j < top; j++) {
                const uint64_t m = __ballot(passes(j));
                row = lane == j ? m : row;
            }
            uint32_t inc = (uint32_t)__popcll(row);
#pragma unroll
            for (int s = 1; s < 64; s <<= 1) {
                const uint32_t y = (uint32_t)__shfl_up((int)inc, s, 64);
                if (lane >= s) inc += y;
            }
            const uint32_t rest = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
            unsigned long long g = 0;
            if (lane == 0) g = atomicAdd(o.counter, (unsigned long long)rest);
            g = (unsigned long long)__shfl((long long)g, 0, 64);
            const uint32_t first = inc - (uint32_t)__popcll(row);
            for (int j = 0; j < top; j++) {
                const uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)row, j) |
                                   ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(row >> 32), j) << 32);
                const int64_t at = (int64_t)g + (uint32_t)__builtin_amdgcn_readlane((int)first, j) +
                                   __popcll(m & ((1ull << lane) - 1));
                if (((m >> lane) & 1ull) && at < o.cap) o.out[at] = pair(j);
            }
        }
        if (++u >= uend) break;
        if (++I > J) {
            I = 0;
            if (++J >= ((uint64_t)z + 63) / 64) {
                J = 0;
                d++;  // every slot has a tile pair
                sl = o.xslot[d];
                loaded = -1;
            }
        }
    }
    if (staged) drain();
}

bool bucket_join_fits(int64_t records, bool members, int64_t total) {
    return records >= 2 && records <= (members ? BK_MEMBERS_MAX : BK_RECORDS_MAX) && total < (1ll << 29);
}

BucketRecords bucket_records(uint64_t *key, uint64_t *val, int64_t cap, int64_t expect, bool members,
                             bool fine, int64_t pass, const int64_t *n_dev, Workspace &ws,
                             hipStream_t s) {
    BucketRecords r;
    r.n = cap;
    r.n_dev = n_dev;
    r.bits = record_bits(expect, members || fine);
    r.key = key;
    r.val = val;
    for (int p = bucket_passes(r.bits); p > 0; p--) {
        uint64_t *ko = ws.get_n<uint64_t>(cap + 1), *vo = ws.get_n<uint64_t>(cap + 1);
        radix_pass(r.key, r.val, ko, vo, cap, 64 - 8 * p, ws, s, n_dev);
        r.key = ko;
        r.val = vo;
    }
    const int64_t nb = 1ll << r.bits;
    // as many workgroups as the device holds at once (their registers leave room for two of 512
    // threads a CU, or four of 256), each with an equal share of the buckets
    r.blocks = (int)(nb <= 256 ? nb
                               : std::min<int64_t>(nb, members ? resident_grid(k_bucket_pairs<true>, BK_MTHREADS)
                                                               : resident_grid(k_bucket_pairs<false>, BK_THREADS)));
    r.members = members;
    // a tile pair of one key has 1,000 tests or more on average; slots of several keys may have
    // fewer, up to this many tile pairs (2^20, about 5 ms, for the default pass)
    r.max_units = (uint64_t)std::max<int64_t>(1024, pass / 256);
    // the workgroups' sums; candidates, over, the long slots' state
    r.state = reinterpret_cast<uint64_t *>(ws.zeroed(6, s));
    r.part = ws.get_n<uint64_t>(3 * r.blocks);
    r.counter = reinterpret_cast<unsigned long long *>(r.state);
    r.over = reinterpret_cast<uint32_t *>(r.state + 1);
    r.dedup_over = r.over + 1;
    r.xcap = cap;
    r.xkey = ws.get_n<uint64_t>(r.xcap + 1);
    r.xrec = reinterpret_cast<int4 *>(ws.get((size_t)(r.xcap + 1) * 16));
    r.xslots = r.xcap / (BK_LONG + 1) + 1;
    r.xslot = reinterpret_cast<ulonglong2 *>(ws.get((size_t)r.xslots * 16));
    r.ustart = ws.get_n<uint64_t>(r.xslots + 1);
    return r;
}

void bucket_reset(const BucketRecords &r, hipStream_t s) { fill_u64(r.state, 0, 3, s); }

void bucket_pairs(const BucketRecords &r, const DevStrings &d, uint64_t *out, int64_t cap, bool longs,
                  hipStream_t s, KTimer *kt) {
    const BucketIn in{r.key, r.val, r.n, r.n_dev, r.bits, d.len, d.kk};
    const BucketOut o{out, cap, r.counter, r.part, r.over, r.xkey, r.xrec, r.xcap, r.xslot, r.xslots,
                      r.counter + 2, r.max_units};
    int th = kt ? kt->begin(KTimer::EMIT, s) : -1;
    hipLaunchKernelGGL((r.members ? k_bucket_pairs<true> : k_bucket_pairs<false>), dim3((unsigned)r.blocks), dim3(r.members ? BK_MTHREADS : BK_THREADS), 0, s, in, o);
    MJ_LAUNCH_CHECK();
    if (longs) {
        hipLaunchKernelGGL(k_long_units, dim3(1), dim3(BK_THREADS), 0, s, r.xslot, r.xslots,
                           r.counter + 2, r.ustart);
        MJ_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_long_pairs, dim3(1024), dim3(64 * LP_WAVES), 0, s, r.ustart, o);
        MJ_LAUNCH_CHECK();
    }
    if (kt) kt->end(th, s);
}

// ---------------------------------------------------------------- dedup
// pairs (first << 32 | second) -> first << b | second; their number (at most cap) to *n_dev
__global__ void k_pack_bucket_pairs(uint64_t *p, const unsigned long long *count, int64_t cap, int b,
                                    int64_t *n_dev) {
    const int64_t n = min(cap, (int64_t)*count);
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_dev = n;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = ((p[i] >> 32) << b) | (p[i] & 0xFFFFFFFFull);
}

// Buckets of equal top `bits` of kb key bits (grouped by them already): each bucket's distinct
// keys by an LDS hash table, sorted there, to uq from the bucket's start on, their number to
// cnt[b].  (Most candidates come several times, some pairs thousands of times: sorting the
// buckets whole took 2.4 ms where one of them held most of 0.5 M candidates of 26 K pairs.)  A
// bucket of more than DD_CAP distinct keys goes by parts of equal further bits, a sweep each, up to
// DD_SWEEP keys swept: pairs of a few neighbouring strings all lie in one bucket, and 1.1 M pairs
// of 1,500 of 60,000 strings took 6.7 ms where sorting them takes 0.2.
// SOLE (one bucket, keys not packed yet): the distinct pairs to uq, their number to *u_dev.
template <bool SOLE>
__global__ __launch_bounds__(BK_THREADS) void k_dedup_buckets(const uint64_t *__restrict__ key,
                                                              const unsigned long long *count,
                                                              int64_t cap, int kb, int bits, int bs,
                                                              uint32_t *__restrict__ cnt,
                                                              uint64_t *__restrict__ uq,
                                                              uint32_t *__restrict__ u_dev,
                                                              uint32_t *__restrict__ over) {
    __shared__ __attribute__((aligned(16))) uint32_t table[2 * DD_CAP];
    __shared__ uint32_t v[DD_CAP];
    __shared__ uint32_t taken;
    __shared__ int64_t bound[2];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t n = min(cap, (int64_t)*count);
    const int shift = kb - bits;
    if (wv < 2) {
        const int64_t b = (int64_t)blockIdx.x + wv;
        const int64_t at = b == 0 ? 0 : b == (1ll << bits) ? n : bucket_start(key, n, shift, (uint64_t)b);
        if (lane == 0) bound[wv] = at;
    }
    __syncthreads();
    const int64_t lo = bound[0], m64 = bound[1] - lo;
    const uint32_t mask = (1u << shift) - 1u;  // shift <= 31: ~0 marks a free entry
    const uint64_t high = SOLE ? 0 : (uint64_t)blockIdx.x << shift;
    const uint64_t low = (1ull << bs) - 1;
    auto entry = [&](int64_t i) -> uint32_t {
        uint64_t x = key[lo + i];
        if (SOLE) x = ((x >> 32) << bs) | (x & 0xFFFFFFFFull);
        return (uint32_t)x & mask;
    };
    if (m64 > DD_SWEEP) {  // (workgroup-uniform)
        if (threadIdx.x == 0) {
            *over = OVER_DEDUP;
            if (SOLE) *u_dev = 0;
            else cnt[blockIdx.x] = 0;
        }
        return;
    }
    int rb = 0;         // 2^rb parts
    uint32_t done = 0;  // distinct keys written
    for (uint32_t part = 0; part < (1u << rb); part++) {
        // the part's distinct keys: open addressing, at most half the table
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * DD_CAP / 4; i += BK_THREADS)
            reinterpret_cast<uint4 *>(table)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
        if (threadIdx.x == 0) taken = 0;
        __syncthreads();
        for (int64_t i0 = threadIdx.x; i0 < m64; i0 += DD_BATCH * BK_THREADS) {
            if (*(volatile uint32_t *)&taken > DD_CAP) break;
            uint32_t xs[DD_BATCH];  // loads in flight together
#pragma unroll
            for (int u = 0; u < DD_BATCH; u++)
                xs[u] = i0 + u * BK_THREADS < m64 ? entry(i0 + u * BK_THREADS) : ~0u;
#pragma unroll
            for (int u = 0; u < DD_BATCH; u++) {
                const uint32_t x = xs[u];
                if (x == ~0u || (rb && (x >> (shift - rb)) != part)) continue;
                for (uint32_t h = (x * 0x9E3779B1u) >> (32 - DD_LOG); ; h = (h + 1) & (2 * DD_CAP - 1)) {
                    uint32_t y = *(volatile uint32_t *)&table[h];
                    if (y == x || *(volatile uint32_t *)&taken > DD_CAP) break;
                    if (y != ~0u) continue;
                    y = atomicCAS(&table[h], ~0u, x);
                    if (y == ~0u) atomicAdd(&taken, 1u);
                    if (y == ~0u || y == x) break;
                }
            }
        }
        __syncthreads();
        const int m = (int)taken;
        if (m > DD_CAP) {
            const int finer = min(min(shift, DD_PARTS), rb + 2);
            if (finer > rb && m64 << finer <= DD_SWEEP) {  // again, by smaller parts
                rb = finer;
                part = ~0u;
                done = 0;
                continue;
            }
            if (threadIdx.x == 0) *over = OVER_DEDUP;
            break;
        }
        if (m == 0) continue;
        __syncthreads();
        if (threadIdx.x == 0) taken = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * DD_CAP; i += BK_THREADS) {
            const uint32_t x = table[i];
            if (x != ~0u) v[atomicAdd(&taken, 1u)] = x;
        }
        int m2 = 64;
        while (m2 < m) m2 <<= 1;
        for (int i = m + threadIdx.x; i < m2; i += BK_THREADS) v[i] = ~0u;
        // bitonic sort; a thread's pairs of a stage of distance < 64 lie in its wave's own
        // 128 entries when the stage before did too, so those need no barrier
        for (int size = 2; size <= m2; size <<= 1) {
            for (int dist = size >> 1; dist > 0; dist >>= 1) {
                if (dist >= 64 || size == 2 || dist == size >> 1) __syncthreads();
                else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                for (int t = threadIdx.x; t < m2 / 2; t += BK_THREADS) {
                    const int i = 2 * t - (t & (dist - 1));
                    const uint32_t a = v[i], b = v[i + dist];
                    const bool up = (i & size) == 0;
                    if ((a > b) == up) {
                        v[i] = b;
                        v[i + dist] = a;
                    }
                }
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < m; i += BK_THREADS) {
            const uint64_t k = high | v[i];
            uq[lo + done + i] = SOLE ? ((k >> bs) << 32) | (k & low) : k;
        }
        done += (uint32_t)m;
    }
    if (threadIdx.x == 0) {
        if (SOLE) *u_dev = done;
        else cnt[blockIdx.x] = done;
    }
}

// The buckets' distinct keys together, as pairs; their number to *u_dev.  pre (nullable): the
// exclusive prefix sums of cnt, else each workgroup adds up those before it.
__global__ __launch_bounds__(256) void k_dedup_gather(const uint64_t *__restrict__ key,
                                                      const uint64_t *__restrict__ uq,
                                                      const unsigned long long *count, int64_t cap,
                                                      int kb, int bits, int bs,
                                                      const uint32_t *__restrict__ cnt,
                                                      const uint32_t *__restrict__ pre,
                                                      uint64_t *__restrict__ res,
                                                      uint32_t *__restrict__ u_dev) {
    __shared__ uint32_t tmp[4];
    __shared__ int64_t start;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t n = min(cap, (int64_t)*count);
    const uint32_t b = blockIdx.x;
    if (wv == 0) {
        const int64_t at = b == 0 ? 0 : bucket_start(key, n, kb - bits, b);
        if (lane == 0) start = at;
    }
    uint32_t before = 0;
    if (!pre) {
        for (uint32_t i = threadIdx.x; i < b; i += 256) before += cnt[i];
        for (int d = 32; d >= 1; d >>= 1) before += (uint32_t)__shfl_down((int)before, d, 64);
        if (lane == 0) tmp[wv] = before;
    }
    __syncthreads();
    before = pre ? pre[b] : tmp[0] + tmp[1] + tmp[2] + tmp[3];
    const uint32_t mine = cnt[b];
    const uint64_t low = (1ull << bs) - 1;
    for (uint32_t i = threadIdx.x; i < mine; i += 256) {
        const uint64_t k = uq[start + i];
        res[before + i] = ((k >> bs) << 32) | (k & low);
    }
    if (b + 1 == gridDim.x && threadIdx.x == 0) *u_dev = before + mine;
}

bool dedup_buckets_fit(int64_t expect, int32_t n_first, int32_t n_second) {
    return dedup_plan(expect, 0, n_first, n_second).fits;
}

const uint32_t *dedup_buckets(uint64_t *pairs, int64_t cap, int64_t expect, int64_t distinct,
                              const unsigned long long *count, int32_t n_first, int32_t n_second,
                              uint32_t *over, Workspace &ws, hipStream_t s, uint64_t **result) {
    cap = std::max<int64_t>(cap, 1);
    const DedupPlan plan = dedup_plan(expect, distinct, n_first, n_second);
    const int bs = plan.bs, kb = plan.kb, bits = plan.bits;
    if (!plan.fits) throw Error(MJ_ECAPACITY, "pairs beyond the dedup's buckets");
    uint64_t *res = ws.get_n<uint64_t>(cap + 1);
    uint32_t *u = ws.get_n<uint32_t>(2);
    *result = res;
    if (bits == 0) {
        hipLaunchKernelGGL(k_dedup_buckets<true>, dim3(1), dim3(BK_THREADS), 0, s, pairs, count, cap,
                           kb, 0, bs, (uint32_t *)nullptr, res, u, over);
        MJ_LAUNCH_CHECK();
        return u;
    }
    int64_t *n_dev = ws.get_n<int64_t>(2);
    hipLaunchKernelGGL(k_pack_bucket_pairs,
                       dim3((unsigned)std::min<int64_t>((cap + 255) / 256, 4096)), dim3(256), 0, s,
                       pairs, count, cap, bs, n_dev);
    MJ_LAUNCH_CHECK();
    uint64_t *k = pairs;
    for (int p = bucket_passes(bits); p > 0; p--) {
        uint64_t *ko = ws.get_n<uint64_t>(cap + 1);
        radix_pass(k, nullptr, ko, nullptr, cap, std::max(0, kb - 8 * p), ws, s, n_dev);
        k = ko;
    }
    uint32_t *cnt = ws.get_n<uint32_t>(1ll << bits);
    uint64_t *uq = ws.get_n<uint64_t>(cap + 1);
    hipLaunchKernelGGL(k_dedup_buckets<false>, dim3(1u << bits), dim3(BK_THREADS), 0, s, k, count,
                       cap, kb, bits, bs, cnt, uq, u, over);
    MJ_LAUNCH_CHECK();
    uint32_t *pre = nullptr;
    if (bits > 10) {
        pre = ws.get_n<uint32_t>((1ll << bits) + 1);
        exclusive_scan_u32(cnt, pre, 1ll << bits, ws, s);
    }
    hipLaunchKernelGGL(k_dedup_gather, dim3(1u << bits), dim3(256), 0, s, k, uq, count, cap, kb, bits,
                       bs, cnt, pre, res, u);
    MJ_LAUNCH_CHECK();
    return u;
}

}  // namespace mj
