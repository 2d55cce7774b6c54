// Batched verification, the skewed band: a pair's band words sit on a ring of lanes, each a
// column behind the lane above it.
//
// As in the column split of verify_lg.hip two halves share a pair, one forward over the
// first half of the text, one over the reversed rest, and meet at the middle column.  In
// each half the pattern is cut into strips of R = 32 W - 1 rows.  Lane w of a ring of G
// lanes holds strip w and works on column t - w at step t, so the horizontal deltas that
// leave the strip above at a column are there one step before they are needed: one DPP row
// rotation each, and no carry has to cross lanes within a column.  (Myers' recurrence takes
// the carry into a word from the delta that enters it: a -1 entering is exactly the carry
// that a longer addition would bring in.)  A strip is needed for the columns at which the
// band meets its rows; then its lane takes the strip G further down.  With R + 1 = P = 32 W
// the strips begin and end at steps congruent to 1 - bhi modulo P once the band reaches
// P c + 1 diagonals below bhi, so all of that happens between blocks of 32 steps.  (c counts
// K, not K - 1: the delta a strip takes in at the last column of the strip above is made up,
// and that cell has to lie outside the true band.)  At a step c + 1 strips are on the ring,
// but up to c + 2 hold rows of the band at the middle column, where they wait: G >= c + 2.
//
// What bounds it: VALU issue, and for few or long pairs the chain of columns (about 20
// instructions a step with one word a lane and 2 planes, 4.4 cycles each).  A lane group's
// window with carry-lookahead (k_verify_persist) takes about 150 a column with 8 lanes of 4
// words, and twice the columns.  Measured in whole calls, ms, that against this: one query
// (a few pairs of up to 10,000 symbols, K to 1,000) 1.96 -> 0.85; an index of 20,000 strings
// built and asked 64 queries 4.83 -> 2.91; verifying 20,011 pairs of 5,000 symbols at K = 150
// 1.13 -> 0.56 (two lanes a pair before); a join of 7,001 reads of 3,000 symbols at K = 101
// 1.25 -> 1.01.
#include "mj_common.h"
#include "verify_common.h"

namespace mj {

// lane i of a row of 16 reads lane i - N (modulo 16)
template <int N>
__device__ __forceinline__ uint32_t row_ror(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + N, 0xF, 0xF, true);
}

// The ring of G lanes: lanes 16 / G apart in a row of 16, so a rotation of the row by that
// stride is a rotation of the ring.
template <int G>
__device__ __forceinline__ int ring_min(int v) {
    if constexpr (G <= 16) v = min(v, (int)row_ror<8>((uint32_t)v));
    if constexpr (G >= 4) v = min(v, (int)row_ror<4>((uint32_t)v));
    if constexpr (G >= 8) v = min(v, (int)row_ror<2>((uint32_t)v));
    if constexpr (G >= 16) v = min(v, (int)row_ror<1>((uint32_t)v));
    return v;
}

// The value of the same lane of the pair's other half (the neighbouring row for G = 16,
// the neighbouring lane otherwise).
template <int G>
__device__ __forceinline__ uint32_t other_half(uint32_t v) {
    if constexpr (G == 16) {
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);  // lane ^ 16
    } else {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);  // lane ^ 1
    }
}

// Rows of a wave's halves: 32 / G pairs of G strips, kept as 16-bit values for the meeting.
template <int W>
struct RingShared {
    uint16_t val[32 * (32 * W - 1)];
    int32_t strip[64];  // the strip each lane's values belong to, -1: none
};

// The pairs order[0 .. n) with G lanes a half and W words a lane, from the sub-queues whose
// counters `next` holds; returns when every sub-queue is dry.
template <int G, int W, int NP, class Shared>
__device__ __forceinline__ void ring_body(const uint64_t *__restrict__ pairs,
                                          const int64_t *__restrict__ order, int64_t n, VSet A,
                                          VSet B, int kmode, uint8_t *__restrict__ flags,
                                          unsigned long long *cells, unsigned long long *next,
                                          Shared &sh) {
    constexpr int STR = 16 / G, R = 32 * W - 1, P = 32 * W;
    constexpr int FAR = 0x3FFFFFFF;
    const int lane = threadIdx.x & 63;
    const int g = (lane & 15) / STR;
    const bool bwd = G == 16 ? (lane & 16) != 0 : (lane & 1) != 0;
    const int leader_lane = G == 16 ? (lane & 32) : G == 8 ? (lane & 48) : (lane & 50);
    // this pair's number in the wave, and the lane of slot 0 of its second half
    const int pslot = G == 16 ? lane >> 5 : G == 8 ? lane >> 4 : (lane >> 4) * 2 + ((lane >> 1) & 1);
    const int bwd0 = G == 16 ? leader_lane + 16 : leader_lane + 1;
    bool active = false, exhausted = false;
    int qj = (int)((blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) % QUEUES);
    int64_t pi = 0, offx = 0, offy = 0;
    const uint32_t *PX = nullptr, *PY = nullptr;
    int32_t K = 0, mp = 0, nt = 0, ncols = 0, bhi = 0, life = 0, band = 0;
    int32_t t0 = 0, tfin = 0;   // next step, last step of this half
    int32_t w = 0, tE = 0;      // this lane's strip and the step after its last
    bool live = false;          // the strip has begun
    int32_t S = 0;              // value at the strip's last row, current column
    int32_t lbsum = 0;          // lower bound of both halves together
    uint32_t Pv[W], Mv[W], PL[W][NP], PLn[W][NP], TY[NP], TYn[NP];
    uint32_t phs = 0, mhb = 0;  // deltas leaving the strip: +1 in bit 31, -1 in bit 0
    uint64_t my_cells = 0;
#pragma unroll
    for (int s = 0; s < W; s++) {
        Pv[s] = Mv[s] = 0;
#pragma unroll
        for (int p = 0; p < NP; p++) PL[s][p] = PLn[s][p] = 0;
    }
#pragma unroll
    for (int p = 0; p < NP; p++) TY[p] = TYn[p] = 0;
    // pattern words s of strip v (rows R v + 32 s + 1 ..), text words from column j on; both
    // reversed in the second half.  A strip that begins meets the band, so it ends at most K +
    // R + 32 symbols past the pattern, and a half's columns end a few strips' steps past its
    // own: within the planes' padding (3,072 symbols), or before their start.
    auto xwords = [&](int v, int s, uint32_t (&o)[NP]) {
        const int64_t at = (int64_t)R * v + 32 * s;
        load_planes<NP>(PX, bwd ? offx + mp - 32 - at : offx + at, bwd, o);
    };
    auto ywords = [&](int j, uint32_t (&o)[NP]) {
        const int64_t at = j - 1;
        load_planes<NP>(PY, bwd ? offy + nt - 32 - at : offy + at, bwd, o);
    };
    for (;;) {
        // ---- pairs whose two halves are done, or rejected: an alignment pays at least the
        // forward bound before the forward lanes' columns and the backward bound after the
        // backward lanes' (disjoint parts of it)
        const bool done = active && t0 > tfin;
        const bool rej = active && lbsum > K;
        const bool odone = other_half<G>(done ? 1u : 0u) != 0u;
        const bool meet = done && odone && !rej;
        if (__any(meet)) {
            // the second half's values by row
            if (bwd && meet) {
                sh.strip[lane] = live ? w : -1;
                uint16_t *v = sh.val + (pslot * G + g) * R;
                int d = S;
#pragma unroll
                for (int s = 0; s < W; s++) d -= __popc(Pv[s] & (s == W - 1 ? 0x7FFFFFFFu : ~0u)) -
                                                 __popc(Mv[s] & (s == W - 1 ? 0x7FFFFFFFu : ~0u));
#pragma unroll
                for (int s = 0; s < W; s++) {
                    const int rows = s == W - 1 ? 31 : 32;
                    for (int b = 0; b < rows; b++) {
                        d += (int)((Pv[s] >> b) & 1u) - (int)((Mv[s] >> b) & 1u);
                        v[32 * s + b] = (uint16_t)min(d, 0xFFFF);
                    }
                }
            }
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
            int best = FAR;
            if (!bwd && meet && live) {
                // row i meets the second half's row mp - i
                auto at_row = [&](int r) -> int {  // r >= 1
                    const int v = (r - 1) / R, sl = v & (G - 1);
                    if (sh.strip[bwd0 + sl * STR] != v) return FAR;
                    return sh.val[(pslot * G + sl) * R + (r - 1 - v * R)];
                };
                const int ncb = nt - ncols;  // the second half's columns
                int d = S;
#pragma unroll
                for (int s = 0; s < W; s++) d -= __popc(Pv[s] & (s == W - 1 ? 0x7FFFFFFFu : ~0u)) -
                                                 __popc(Mv[s] & (s == W - 1 ? 0x7FFFFFFFu : ~0u));
                if (w == 0) best = ncols + at_row(mp);  // row 0
                const int rt = mp - R * w - 1;          // the partner of the strip's first row
                int va = rt >= 1 ? (rt - 1) / R : 0;
                int ba = rt - 1 - va * R;               // its place in its strip
                int sl = va & (G - 1);
                bool ok = sh.strip[bwd0 + sl * STR] == va;
                const uint16_t *vp = sh.val + (pslot * G + sl) * R;
#pragma unroll
                for (int s = 0; s < W; s++) {
                    const int rows = s == W - 1 ? 31 : 32;
                    for (int b = 0; b < rows; b++) {
                        const int r = rt - 32 * s - b;  // the partner row
                        d += (int)((Pv[s] >> b) & 1u) - (int)((Mv[s] >> b) & 1u);
                        if (r < 0) break;
                        if (r == 0) {
                            best = min(best, d + ncb);
                            break;
                        }
                        if (ba < 0) {  // the strip above
                            va--;
                            ba = R - 1;
                            sl = va & (G - 1);
                            ok = sh.strip[bwd0 + sl * STR] == va;
                            vp = sh.val + (pslot * G + sl) * R;
                        }
                        if (ok) best = min(best, d + (int)vp[ba]);
                        ba--;
                    }
                }
            }
            best = ring_min<G>(best);
            if (meet && lane == leader_lane) flags[pi] = best <= K ? 1 : 0;
            __builtin_amdgcn_wave_barrier();
        }
        if (rej && lane == leader_lane) flags[pi] = 0;
        if (rej || meet) active = live = false;

        // ---- refill: each pair slot without a pair takes the next one
        const bool need = !active && !exhausted;
        const long long got = __shfl(take_pairs(next, n, need && lane == leader_lane, qj, exhausted), leader_lane, 64);
        if (need && got >= 0 && got < n) {
            pi = order[got];
            const uint64_t pr = pairs[pi];
            const int32_t ia = (int32_t)(pr >> 32), ib = (int32_t)(uint32_t)pr;
            const int32_t ma = A.len[ia], mb = B.len[ib];
            K = kmode == 0 ? max(A.kk[ia], B.kk[ib]) : A.kk[ia];
            const bool a_is_x = ma >= mb;
            PX = a_is_x ? A.planes : B.planes;
            PY = a_is_x ? B.planes : A.planes;
            offx = a_is_x ? A.off[ia] : B.off[ib];
            offy = a_is_x ? B.off[ib] : A.off[ia];
            mp = a_is_x ? ma : mb;
            nt = a_is_x ? mb : ma;
            const int dlen = mp - nt;
            const int blo = -((K - dlen) >> 1);  // band diagonals blo .. bhi
            bhi = (K + dlen) >> 1;
            band = bhi - blo + 1;
            const int c = (bhi - blo + P - 1) / P;
            uint8_t result = 0;
            bool trivial = true;
            if (dlen > K) {
                result = 0;
            } else if (nt == 0) {
                result = mp <= K;
            } else if (c + 2 > G) {
                result = 2;
            } else {
                trivial = false;
            }
            if (trivial) {
                if (lane == leader_lane) flags[pi] = result;
                if (lane == leader_lane && result == 2) atomicOr(cells + 1, 1ull);
            } else {
                active = true;
                const int mid = nt >> 1;
                ncols = bwd ? nt - mid : mid;
                life = P * (c + 1);
                // strips begin at steps P w + 1 - bhi; those at or before the first step
                // (the last boundary not after step 1) have begun
                const int skip = bhi % P;
                t0 = 1 - (skip & 31);
                w = g;
                live = g <= bhi / P;
                tE = P * w + 1 - bhi + life;
                tfin = ncols + min(mp - 1, max(ncols + bhi - 1, 0)) / R;
                S = R * w + R;  // column 0: row i holds i
                lbsum = 0;
                phs = mhb = 0;
                ywords(t0 - w, TY);
#pragma unroll
                for (int s = 0; s < W; s++) {
                    Pv[s] = ~0u;
                    Mv[s] = 0u;
                    if (live) xwords(w, s, PL[s]);
                }
            }
        }
        if (__all(!active && exhausted)) break;

        // ---- the next block's text words and, for a lane that begins a strip then, its
        // pattern words (loads in flight over this block)
        const int tn = t0 + 32;
        // a strip that ends before the half's last column makes room for the one G further
        const bool adv = active && live && tn == tE && tn - 1 - w < ncols;
        const int wn = adv ? w + G : w;
        const int tEn = adv ? tE + P * G : tE;
        const bool begin = active && (adv || !live) && tn == tEn - life && tn - wn <= ncols;
        if (active) ywords(tn - wn, TYn);
        if (begin) {
#pragma unroll
            for (int s = 0; s < W; s++) xwords(wn, s, PLn[s]);
        }

        // ---- 32 steps
        const int j0 = t0 - w;  // this lane's first column
        // the deltas entering the top strip: +1 a column (its upper neighbour is outside the
        // band, or row 0)
        const bool top = w == 0 || t0 >= tE - P;
        const uint32_t topm = top ? 0x80000000u : 0u, ntop = top ? 0u : 1u;
        uint32_t accP = 0;
        auto step = [&](uint32_t tb[NP], uint32_t (&nP)[W], uint32_t (&nM)[W], uint32_t &nph,
                        uint32_t &nmh) {
            const uint32_t hb = row_ror<STR>(mhb) & ntop;
            uint32_t pin = row_ror<STR>(phs) | topm;
            uint32_t eq[W], xh[W];
#pragma unroll
            for (int s = 0; s < W; s++) {
                uint32_t e = ~(PL[s][0] ^ tb[0]);
#pragma unroll
                for (int p = 1; p < NP; p++) e = and_xnor(e, PL[s][p], tb[p]);
                eq[s] = e;
            }
            if constexpr (W == 1) {
                const uint32_t x = eq[0] & Pv[0];
                const uint32_t sum = x + Pv[0] + hb;
                xh[0] = (sum ^ Pv[0]) | eq[0];
            } else {
                uint32_t carry = 0;
#pragma unroll
                for (int s = 0; s < W; s++) {
                    const uint32_t e = s == 0 ? eq[0] | hb : eq[s];
                    uint32_t co;
                    const uint32_t sum = __builtin_addc(e & Pv[s], Pv[s], carry, &co);
                    carry = co;
                    xh[s] = (sum ^ Pv[s]) | e;
                }
            }
            uint32_t mlow = hb, mprev = 0;
#pragma unroll
            for (int s = 0; s < W; s++) {
                const uint32_t ph = Mv[s] | ~(xh[s] | Pv[s]);
                const uint32_t mh = Pv[s] & xh[s];
                const uint32_t phl = __builtin_amdgcn_alignbit(ph, pin, 31);
                const uint32_t mhl = s == 0 ? (mh << 1) | mlow : __builtin_amdgcn_alignbit(mh, mprev, 31);
                const uint32_t xv = eq[s] | Mv[s];
                nP[s] = mhl | ~(xv | phl);
                nM[s] = phl & xv;
                pin = ph;
                mprev = mh;
                if (s == W - 1) {
                    nph = phl;                  // bit 31: row R's delta is +1
                    nmh = (mh >> 30) & 1u;      // row R's delta is -1
                }
            }
        };
        const bool edge = live && (j0 < 1 || j0 + 31 > ncols);
        if (!__any(edge)) {
#pragma unroll 1
            for (int u = 0; u < 4; u++) {
#pragma unroll
                for (int t = 0; t < 8; t++) {
                    uint32_t tb[NP];
#pragma unroll
                    for (int p = 0; p < NP; p++) tb[p] = (uint32_t)__builtin_amdgcn_sbfe((int)TY[p], t, 1u);
                    step(tb, Pv, Mv, phs, mhb);
                    accP = __builtin_amdgcn_alignbit(accP, phs, 31);
                    S -= (int)mhb;
                }
#pragma unroll
                for (int p = 0; p < NP; p++) TY[p] >>= 8;
            }
        } else {
            // columns before the first and after the half's last leave a lane as it is
#pragma unroll 1
            for (int t = 0; t < 32; t++) {
                uint32_t tb[NP];
#pragma unroll
                for (int p = 0; p < NP; p++) {
                    tb[p] = (uint32_t)((int)(TY[p] << 31) >> 31);
                    TY[p] >>= 1;
                }
                const bool in = (uint32_t)(j0 + t - 1) < (uint32_t)ncols;
                uint32_t nP[W], nM[W], nph, nmh;
                step(tb, nP, nM, nph, nmh);
#pragma unroll
                for (int s = 0; s < W; s++) {
                    Pv[s] = in ? nP[s] : Pv[s];
                    Mv[s] = in ? nM[s] : Mv[s];
                }
                phs = in ? nph : phs;
                mhb = in ? nmh : mhb;
                accP = (accP << 1) | (in ? nph >> 31 : 0u);
                S -= in ? (int)nmh : 0;
            }
        }
        S += __popc(accP);
        if (active && g == 0)
            my_cells += (uint64_t)(min(ncols, tn - 1) - min(ncols, max(t0 - 1, 0))) * (uint64_t)band;
        t0 = tn;
        // ---- a lower bound of what any alignment pays before it leaves the columns done:
        // the least value of the strips' current columns, less one at a strip's last row
        // (an alignment may leave it one column earlier, into the strip below)
        {
            int bot = S, lb = FAR;
#pragma unroll
            for (int s = W - 1; s >= 0; s--) {
                const uint32_t m = s == W - 1 ? 0x7FFFFFFFu : ~0u;
                const int pp = __popc(Pv[s] & m);
                lb = min(lb, bot - pp);
                bot += __popc(Mv[s] & m) - pp;
            }
            lb = min(lb, S - 1);
            lb = ring_min<G>(live ? lb : FAR);
            lbsum = lb + (int)other_half<G>((uint32_t)lb);
        }
        // ---- strips that end and begin.  A new strip's values hang below the strip above,
        // one column back: rows one apart
        const int above = (int)row_ror<STR>((uint32_t)(S - (int)(phs >> 31) + (int)mhb));
        if (adv) {
            w = wn;
            tE = tEn;
            live = false;
        }
        if (begin) {
            live = true;
            S = above + R;
#pragma unroll
            for (int s = 0; s < W; s++) {
                Pv[s] = ~0u;
                Mv[s] = 0u;
#pragma unroll
                for (int p = 0; p < NP; p++) PL[s][p] = PLn[s][p];
            }
        }
#pragma unroll
        for (int p = 0; p < NP; p++) TY[p] = TYn[p];
    }
    for (int d = 32; d >= 1; d >>= 1) {
        uint32_t lo = (uint32_t)my_cells, hi = (uint32_t)(my_cells >> 32);
        lo = __shfl_down(lo, d, 64);
        hi = __shfl_down(hi, d, 64);
        my_cells += ((uint64_t)hi << 32) | lo;
    }
    if (lane == 0 && my_cells) atomicAdd(cells, (unsigned long long)my_cells);
}

// One persistent launch over the classes 0 .. CMAX of ring_class, the widest bands first.  The
// wide classes' registers (W words of each of NP planes, twice) leave two waves a SIMD: calls
// without such bands take a kernel without them.
template <int NP, int CMAX>
__global__ __launch_bounds__(256) void k_verify_ring(const uint64_t *__restrict__ pairs,
                                                     const int64_t *__restrict__ order,
                                                     const uint32_t *__restrict__ off, VSet A,
                                                     VSet B, int kmode,
                                                     uint8_t *__restrict__ flags,
                                                     unsigned long long *cells,
                                                     unsigned long long *next) {
    __shared__ RingShared<RING_W[CMAX]> shared[4];
    auto &sh = shared[threadIdx.x >> 6];
    for (int c = CMAX; c >= 0; c--) {
        const int b0 = (RING_CLASSES - 1 - c) * RING_BINS;
        const int64_t base = off[b0], cnt = (int64_t)off[b0 + RING_BINS] - base;
        if (cnt <= 0) continue;
        unsigned long long *nx = next + (int64_t)c * QUEUES * QSTRIDE;
        const int64_t *oc = order + base;
        switch (c) {
            case 0: ring_body<4, 1, NP>(pairs, oc, cnt, A, B, kmode, flags, cells, nx, sh); break;
            case 1: ring_body<8, 1, NP>(pairs, oc, cnt, A, B, kmode, flags, cells, nx, sh); break;
            case 2: ring_body<16, 1, NP>(pairs, oc, cnt, A, B, kmode, flags, cells, nx, sh); break;
            case 3:
                if constexpr (CMAX >= 3)
                    ring_body<16, 2, NP>(pairs, oc, cnt, A, B, kmode, flags, cells, nx, sh);
                break;
            case 4:
                if constexpr (CMAX >= 4)
                    ring_body<16, 3, NP>(pairs, oc, cnt, A, B, kmode, flags, cells, nx, sh);
                break;
            default:
                if constexpr (CMAX >= 5)
                    ring_body<16, 5, NP>(pairs, oc, cnt, A, B, kmode, flags, cells, nx, sh);
                break;
        }
    }
}

template <int NP>
static PersistClassKernel ring_by_class(int c) {
    return c <= 2 ? k_verify_ring<NP, 2> : c == 3 ? k_verify_ring<NP, 3>
         : c == 4 ? k_verify_ring<NP, 4> : k_verify_ring<NP, 5>;
}

PersistClassKernel ring_kernel(int np, int cmax) {
    const int c = ring_class(32 * cmax);
    switch (np) {
        case 2: return ring_by_class<2>(c);
        case 4: return ring_by_class<4>(c);
        case 6: return ring_by_class<6>(c);
        default: return ring_by_class<8>(c);
    }
}

}  // namespace mj
