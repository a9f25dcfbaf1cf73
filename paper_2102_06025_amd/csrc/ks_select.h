// Internal interface of the selection stage (see ks_select.hip), and the device code of the single-workgroup selection,
// which also runs as extra workgroups of the step's own launches (the selection of the NEXT batch, ks_softmax.hip).
#pragma once
#include <type_traits>
#include "ks_common.h"

size_t ks_select_ws_bytes(int64_t C, int B, int K);
// Enqueues the selection kernels on `st`.  Arguments must already be validated.
int ks_select_launch(const int32_t *labels, const int32_t *graph, int64_t C, int B, int K, int M,
                     int32_t *active_idx, int32_t *n_active, int32_t *target_pos, void *ws,
                     int32_t *dev_status, hipStream_t st);

#define SEL1_WS_CLASSES 393216 /* up to this many classes the workspace is sized for the staged candidates, beyond for the score table */
#define SEL1_NT 1024
#define SEL1_GRID 32
#define SEL1_FIRST_WORDS 257 /* one bit per sample of batches up to 8,192 (+ one word so that a clear loop may run over) */
#define SEL1_LDS_WORDS 40600 /* LDS of the single-workgroup selection (162,400 of 163,840 bytes) */
#define SEL1_FIXED_WORDS 540 /* first-of-its-label bits (257), digit counts (256), block scan (1024 / 64 + 1), five scalars, to a multiple of 4 */
#define SEL1_WALK 8          /* list positions that the search of the cut takes one by one (see sel1_body) */
// The selection by one workgroup needs LDS for a bit per class, the running count at every 32nd word of them, and (when the
// cut bites) the classes first seen at the cut position, at most one per sample and per class.
__host__ __device__ __forceinline__ bool sel1_fits(int64_t C, int B) {
    const int64_t nq = (C + 1023) >> 10, n_list = B < C ? B : C;
    return nq * 33 + n_list + SEL1_FIXED_WORDS <= SEL1_LDS_WORDS;
}

// candidate at list position r of sample i (r = 0: the sample's own class), as an id in [0, C), or -1
struct SelDense {
    const int32_t *labels, *graph;
    int64_t C;
    int K;
    static constexpr bool kForeignLabels = false; // a label this GPU does not own is an error
    __device__ __forceinline__ int32_t cand(int i, int r, int32_t *dev_status) const {
        const int32_t y = labels[i];
        if (y < 0 || y >= C) {
            if (r == 0) ks_flag(dev_status, KS_DEV_BAD_LABEL);
            return -1;
        }
        if (r == 0) return y;
        int32_t c = graph[(int64_t)y * K + (r - 1)];
        if (c < -1 || c >= C) {
            ks_flag(dev_status, KS_DEV_BAD_GRAPH_ID);
            c = -1;
        }
        return c;
    }
};
struct SelCsr {
    const int32_t *labels, *counts;
    const int64_t *offsets;
    const int32_t *flat;
    int64_t Cg, c0, C, flat_len; // classes of the whole problem; first class and number of classes of this node
    int K;                       // upper bound of the list lengths
    static constexpr bool kForeignLabels = true; // labels of other nodes' classes have no target here
    __device__ __forceinline__ int32_t cand(int i, int r, int32_t *dev_status) const {
        const int32_t y = labels[i];
        if (y < 0 || y >= Cg) {
            if (r == 0) ks_flag(dev_status, KS_DEV_BAD_LABEL);
            return -1;
        }
        if (r == 0) {
            const int64_t l = (int64_t)y - c0;
            return (l >= 0 && l < C) ? (int32_t)l : -1;
        }
        const int32_t n = counts[y];
        if (r - 1 >= n) return -1;
        const int64_t off = offsets[y];
        if (n > K || off < 0 || off + n > flat_len) { // a list longer than promised or outside the array: not read
            if (r == 1) ks_flag(dev_status, KS_DEV_BAD_COUNT);
            return -1;
        }
        int32_t c = flat[off + (r - 1)];
        if (c < -1 || c >= C) {
            ks_flag(dev_status, KS_DEV_BAD_GRAPH_ID);
            c = -1;
        }
        return c;
    }
};

// k-th draw of the random fill-up: a keyed one-to-one map of [0, 2^b) onto itself (adding a constant, multiplying
// by an odd constant and xor with a right shift of itself are each one-to-one on b-bit numbers), 2^b the smallest
// power of two >= C.  Draws >= C or already in the set are passed over: a sample without replacement of the
// classes not chosen (Algorithm 1 only says "random sample").
struct SelPad {
    int on, b;
    uint32_t mask, s_lo, s_hi;
};
inline SelPad sel_pad_make(int on, int64_t C, uint64_t seed) {
    SelPad p;
    p.on = on;
    p.b = 1;
    while (((int64_t)1 << p.b) < C) ++p.b;
    p.mask = p.b >= 32 ? 0xFFFFFFFFu : ((1u << p.b) - 1u);
    p.s_lo = (uint32_t)seed;
    p.s_hi = (uint32_t)(seed >> 32);
    return p;
}
__device__ __forceinline__ uint32_t sel_pad_draw(uint32_t k, const SelPad &p) {
    const int s1 = (p.b + 1) >> 1, s2 = p.b / 3 > 0 ? p.b / 3 : 1;
    uint32_t x = (k + p.s_lo) & p.mask;
    x = (x * 0x9E3779B1u) & p.mask;
    x ^= x >> s1;
    x = (x * 0x85EBCA6Bu) & p.mask;
    x ^= x >> s2;
    x = (x * 0xC2B2AE35u) & p.mask;
    x ^= x >> s1;
    return (x + p.s_hi) & p.mask;
}

// Number of set bits of the bitmap of 32 nq words; coarse[q] = number of set bits in words < 32 q.  Eight lanes add up
// the 32 words of an entry, four words a lane.
template <int NT>
__device__ __forceinline__ int sel1_count(const uint32_t *bm, int nq, int *coarse, int *sh) {
    const int lane8 = threadIdx.x & 7;
    for (int q0 = 0; q0 < nq; q0 += NT / 8) {
        const int q = q0 + (int)(threadIdx.x >> 3);
        int n = 0;
        if (q < nq) {
            const uint4 v = *(const uint4 *)(bm + q * 32 + lane8 * 4);
            n = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
        }
        n += KS_DPP(0, n, 0x111, 0xf);
        n += KS_DPP(0, n, 0x112, 0xf);
        n += KS_DPP(0, n, 0x114, 0xf); // the last of eight lanes has their sum (others of the row of 16 wrong ones)
        if (lane8 == 7 && q < nq) coarse[q] = n;
    }
    __syncthreads();
    int carry = 0;
    for (int q0 = 0; q0 < nq; q0 += NT) {
        const int q = q0 + (int)threadIdx.x;
        int total;
        const int ex = ks_block_escan<NT>(q < nq ? coarse[q] : 0, sh, &total);
        if (q < nq) coarse[q] = carry + ex;
        carry += total;
    }
    __syncthreads();
    return carry;
}
// Number of set bits alone.
template <int NT> __device__ __forceinline__ int sel1_total(const uint32_t *bm, int nq, int *sh) {
    int n = 0;
    for (int p = threadIdx.x; p < nq * 8; p += NT) {
        const uint4 v = *(const uint4 *)(bm + p * 4);
        n += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
    int total;
    ks_block_escan<NT>(n, sh, &total);
    return total;
}

template <int NT> __device__ __forceinline__ void sel1_clear(uint32_t *bm, int nq) {
    for (int p = threadIdx.x; p < nq * 8; p += NT) *(uint4 *)(bm + p * 4) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
}

// Candidates of a batch as the selection reads them.  mark(r, n, f): f(class) for every candidate at a list position
// in [r, n), possibly for some below r too; at(r, f): for those at position r; label(i): the sample's own class, or -1.
//
// Staged: the candidates lie in memory, list-position-major (cand[r * B + i]), written by an earlier launch: the scattered
// reads of many lists are spread over the chip.
template <int NT> struct Sel1Staged {
    const int32_t *__restrict__ cand;
    int B, K;
    const uint32_t *first; // bit i: sample i is the first of its label (nullptr: not known, all are taken)
    template <class F> __device__ __forceinline__ void range(int64_t begin, int64_t end, F f) const {
        const int tid = threadIdx.x;
        const int64_t n_vec = end >> 2; // (from begin / 4 on; the array is 256-byte aligned: whole pieces, then a tail)
        for (int64_t t0 = begin >> 2; t0 < n_vec; t0 += (int64_t)NT * 8) {
            int4 c[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) { // many loads in flight: the round trips to L2 are what this costs
                const int64_t t = t0 + (int64_t)e * NT + tid;
                c[e] = t < n_vec ? ((const int4 *)cand)[t] : make_int4(-1, -1, -1, -1);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t f4 = 0xFu; // which of the four samples are the first of their label (B a power of two)
                if (first) {
                    const int i0 = (int)(((t0 + (int64_t)e * NT + tid) << 2) & (B - 1));
                    f4 = first[i0 >> 5] >> (i0 & 31);
                }
                if (c[e].x >= 0 && (f4 & 1u)) f(c[e].x);
                if (c[e].y >= 0 && (f4 & 2u)) f(c[e].y);
                if (c[e].z >= 0 && (f4 & 4u)) f(c[e].z);
                if (c[e].w >= 0 && (f4 & 8u)) f(c[e].w);
            }
        }
        for (int64_t t = (n_vec * 4 > begin ? n_vec * 4 : begin) + tid; t < end; t += NT) {
            const int32_t c = cand[t];
            if (c >= 0) f(c);
        }
    }
    template <class F> __device__ __forceinline__ void mark(int r, int n, F f) const { range((int64_t)r * B, (int64_t)n * B, f); }
    template <class F> __device__ __forceinline__ void at(int r, F f) const {
        for (int i0 = 0; i0 < B; i0 += NT * 4) {
            int32_t c[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = i0 + e * NT + (int)threadIdx.x;
                c[e] = i < B ? cand[(int64_t)r * B + i] : -1;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c[e] >= 0) f(c[e]);
        }
    }
    __device__ __forceinline__ int32_t label(int i) const { return cand[i]; }
};
// Direct: batches of at most NT * E candidates are read from the labels and lists by the selecting workgroups themselves
// (every one of them reads all) and stay in registers: one launch instead of two, and the passes of the cut read nothing.
template <int NT, int E, class Src> struct Sel1Direct {
    Src src;
    int32_t c[E];
    int r[E];
    __device__ __forceinline__ void load(int B, int K, bool report, int32_t *dev_status) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int q = e * NT + (int)threadIdx.x;
            const int i = q / (K + 1);
            r[e] = q - i * (K + 1);
            c[e] = i < B ? src.cand(i, r[e], report ? dev_status : nullptr) : -1;
        }
    }
    template <class F> __device__ __forceinline__ void mark(int, int n, F f) const {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (c[e] >= 0 && r[e] < n) f(c[e]);
    }
    template <class F> __device__ __forceinline__ void at(int rr, F f) const {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (c[e] >= 0 && r[e] == rr) f(c[e]);
    }
    __device__ __forceinline__ int32_t label(int i) const { return src.cand(i, 0, nullptr); }
};

// The whole selection by one workgroup of NT threads (see ks_select.hip for the method).  `lds` has SEL1_LDS_WORDS
// words.  The G workgroups that call this with g = 0 .. G - 1 all do the same LDS work and write a G-th of the outputs
// each.  A __device__ function so that the workgroups may be those of a kernel of their own or extra workgroups of
// another launch.
template <int NT, class Cands>
__device__ __forceinline__ void sel1_body(uint32_t *lds, Cands &cands, int64_t C, int B, int K, int M,
                                          int foreign_labels, SelPad pad, int32_t *__restrict__ active_idx,
                                          int32_t *__restrict__ n_active, int32_t *__restrict__ n_found,
                                          int32_t *__restrict__ target_pos, const int G, const int g) {
    const int nq = (int)((C + 1023) >> 10), n_list = B < C ? B : (int)C; // the bitmap has 32 nq words
    const int tid = threadIdx.x;
    uint32_t *s_first = lds;
    int *hist = (int *)(s_first + SEL1_FIRST_WORDS), *sh = hist + 256; // sh: the block scan, then scalars
    int *const s_new = sh + 1024 / 64 + 1, &s_bin = s_new[3], &s_rem = s_new[4];
    uint32_t *bm = lds + SEL1_FIXED_WORDS;
    int *coarse = (int *)(bm + nq * 32), *list = coarse + nq;
    auto bit_of = [&](int32_t c) { return 1u << (c & 31); };
    auto set = [&](int32_t c) { atomicOr(&bm[c >> 5], bit_of(c)); };
    sel1_clear<NT>(bm, nq);
    // Optimistic pass: every candidate, whatever its list position.  Samples with the same label have the same list, and
    // with skewed labels half of the batch are repeats: in the staged form only the first sample of a label (whichever
    // thread marks the label first) has its list marked.  For batch sizes that are a power of two, so that a 16-byte piece
    // of the staging array holds four samples of one list position and the sample index is a mask away.
    if constexpr (std::is_same<Cands, Sel1Staged<NT>>::value) {
        const bool dedup = B >= 4 && (B & (B - 1)) == 0 && B <= SEL1_FIRST_WORDS * 32;
        if (dedup) {
            for (int w = tid; w < B / 32 + 1; w += NT) s_first[w] = 0u;
            __syncthreads();
            for (int i = tid; i < B; i += NT) {
                const int32_t c = cands.label(i); // (-1: a class of another node, whose list still counts)
                bool first = true;
                if (c >= 0) first = !(atomicOr(&bm[c >> 5], bit_of(c)) & bit_of(c));
                if (first) atomicOr(&s_first[i >> 5], 1u << (i & 31));
            }
            __syncthreads();
            cands.first = s_first;
        }
        cands.range(dedup ? B : 0, (int64_t)B * (K + 1), set); // (deduplicated: the labels are done)
    } else {
        cands.mark(0, K + 1, set);
    }
    __syncthreads();
    int total = sel1_count<NT>(bm, nq, coarse, sh);
    if (total > M) {
        // The cut bites.  r* = the first list position up to which more than M classes are seen, between positions known to see
        // at most M (lo) and more (hi).  Two kinds of step, on a bitmap that holds what is seen up to `built`:
        //   probe  mark the candidates of the positions up to another one and count the bits: first, while that is far, the
        //          last position up to which all candidates together cannot bring more than M classes, then an interpolated
        //          guess and a halving in turn.  Costs a pass over those candidates and one over the bitmap; where there
        //          are more than M the bitmap is cleared and built anew up to lo.
        //   walk   position by position from lo on; the classes that are new go into a list.  Costs a read of B candidates
        //          and a barrier, and where it ends at r*, bitmap and list are what the rest needs.
        // Walks are taken where the guess (too high where counts flatten out, as they do) lies within SEL1_WALK positions.
        // 20,000 classes, 1,024 lists of 32, M = 4,096 (r* = 4): position by position 22 us in all, with halvings and guesses on a
        // cleared bitmap 27, so 22.  1,100,000 classes, 2,048 lists of 64, r* in their middle: 64 us -> 40 (26 without a cut).
        int lo = -1, hi = K, n_lo = 0, n_hi = total, built = -1;
        int ctr = 0; // of three counters of the list, this position's: it is cleared while the one before is in use
        bool walked = false;
        sel1_clear<NT>(bm, nq);
        for (int step = 0;; ++step) {
            int mid = lo + 1 + (int)((int64_t)(M - n_lo) * (hi - lo - 1) / (n_hi - n_lo));
            if (hi - lo > SEL1_WALK && (walked || mid - lo > SEL1_WALK)) {
                const int sure = lo + (M - n_lo) / B; // (below hi: that many positions bring no more than M classes)
                if (step < 3 && sure - lo > 2) mid = sure;
                else if (walked || (step & 1)) mid = (lo + hi) >> 1;
                if (mid > hi - 1) mid = hi - 1;
                walked = false;
                cands.mark(built + 1, mid + 1, set);
                __syncthreads();
                const int n = sel1_total<NT>(bm, nq, sh);
                if (n > M) {
                    hi = mid;
                    n_hi = n;
                    built = -1;
                    sel1_clear<NT>(bm, nq);
                } else {
                    lo = built = mid;
                    n_lo = n;
                }
                continue;
            }
            if (built != lo) cands.mark(built + 1, lo + 1, set);
            walked = true;
            if (tid == 0) s_new[ctr] = 0;
            __syncthreads();
            const int end = hi - lo > SEL1_WALK ? lo + SEL1_WALK : hi;
            int r = lo + 1;
            for (;; ++r) {
                cands.at(r, [&](int32_t c) {
                    if (!(atomicOr(&bm[c >> 5], bit_of(c)) & bit_of(c))) {
                        const uint64_t act = __ballot(1);
                        const int before = __popcll(act & ((1ull << (tid & 63)) - 1ull));
                        int slot = 0;
                        if (before == 0) slot = atomicAdd(&s_new[ctr], __popcll(act));
                        slot = __builtin_amdgcn_readfirstlane(slot) + before;
                        if (slot < n_list) list[slot] = c; // always true: a class once, and at most one per sample
                    }
                });
                const int next = ctr == 2 ? 0 : ctr + 1;
                if (tid == 0) s_new[next] = 0; // (read last two positions ago)
                __syncthreads();
                const int n = n_lo + s_new[ctr];
                if (n > M) { hi = r; break; }
                n_lo = n;
                lo = built = r;
                ctr = next;
                if (r == end) break;
            }
            if (hi == lo + 1 && r == hi) break; // ended at r* = hi
        }
        // the classes first seen at r* are in the bitmap and in the list; the M - n_lo lowest ids of them stay
        const int n_new = s_new[ctr] < n_list ? s_new[ctr] : n_list;
        int rem = M - n_lo;       // the rem-th smallest of the list is the last to stay
        uint32_t top = 0u;        // its leading digits so far
        int bits = 32 - __builtin_clz((uint32_t)(C > 1 ? C - 1 : 1)); // not yet looked at, eight at a time from the top
        while (rem > 0 && bits > 0) {
            const int shift = bits > 8 ? bits - 8 : 0;
            for (int q = tid; q < 256; q += NT) hist[q] = 0;
            __syncthreads();
            for (int q = tid; q < n_new; q += NT) {
                const uint32_t c = (uint32_t)list[q];
                if (c >> bits == top >> bits) atomicAdd(&hist[(c >> shift) & ((1u << (bits - shift)) - 1u)], 1);
            }
            __syncthreads();
            if (tid < 64) { // one wavefront: four digits a lane
                int v[4], sum = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[e] = hist[tid * 4 + e]; sum += v[e]; }
                int run = ks_wave_iscan(sum) - sum;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (run < rem && run + v[e] >= rem) { s_bin = tid * 4 + e; s_rem = rem - run; }
                    run += v[e];
                }
            }
            __syncthreads();
            top |= (uint32_t)s_bin << shift;
            rem = s_rem;
            bits = shift;
            __syncthreads();
        }
        const bool none = M == n_lo; // nothing of r* stays
        for (int q = tid; q < n_new; q += NT) {
            const int32_t c = list[q];
            if (none || (uint32_t)c > top) atomicAnd(&bm[c >> 5], ~bit_of(c));
        }
        __syncthreads();
        total = sel1_count<NT>(bm, nq, coarse, sh);
    }
    const int found = total < M ? total : M;
    const int64_t want = M < C ? M : C;
    if (pad.on && total < want) {
        // random fill-up: the first draws that are classes of this GPU and not in the bitmap yet (the draws are
        // distinct, so marking one cannot change the test of another)
        const int need = (int)(want - total);
        const uint32_t n_draws = 1u << pad.b; // b <= 21 here
        int got = 0;
        for (uint32_t k0 = 0; got < need && k0 < n_draws; k0 += NT * 8) {
            uint32_t cs[8];
            int valid = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t k = k0 + (uint32_t)tid * 8 + e;
                const uint32_t c = k < n_draws ? sel_pad_draw(k, pad) : 0xFFFFFFFFu;
                cs[e] = (c < (uint64_t)C && !(bm[c >> 5] & (1u << (c & 31)))) ? c : 0xFFFFFFFFu;
                valid += cs[e] != 0xFFFFFFFFu;
            }
            int tot;
            int ex = ks_block_escan<NT>(valid, sh, &tot);
            const int room = need - got;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (cs[e] != 0xFFFFFFFFu) {
                    if (ex < room) atomicOr(&bm[cs[e] >> 5], 1u << (cs[e] & 31));
                    ++ex;
                }
            got += tot < room ? tot : room;
            __syncthreads();
        }
        total = sel1_count<NT>(bm, nq, coarse, sh);
    }
    // Every workgroup of the grid has built the same bitmap and counts (redundantly: it is LDS work, and it
    // spares a grid-wide synchronisation); each writes its share of the outputs.
    { // read the bitmap out in ascending order: a wavefront takes 64 words, a lane one of them
        const int lane = tid & 63, ngrp = (nq + 1) >> 1;
        // (neighbouring groups on different workgroups: 100,000 classes, all active, are 49 groups)
        for (int q = (tid >> 6) * G + g; q < ngrp; q += G * (NT / 64)) {
            const int w = q * 64 + lane;
            const bool in = w < nq * 32;
            uint32_t e = in ? bm[w] : 0u;
            const int n = __popc(e);
            const int ex = ks_wave_iscan(n) - n, half = __builtin_amdgcn_readlane(ex, 32); // a coarse entry per 32 words
            int pos = in ? coarse[w >> 5] + ex - (lane < 32 ? 0 : half) : 0;
            while (e) {
                const int b = __ffs(e) - 1;
                if (pos < M) active_idx[pos] = w * 32 + b; // pos < M always holds; the test keeps the store in bounds
                ++pos;
                e &= e - 1;
            }
        }
    }
    const int n = total < M ? total : M;
    for (int a = n + g * NT + tid; a < M; a += G * NT) active_idx[a] = -1;
    const int none = foreign_labels ? -1 : 0; // in range even for broken inputs (those are flagged)
    // a half-wave per sample: each lane counts one of the 32 words that share the label's coarse entry
    for (int i0 = (g * (NT / 64) + (tid >> 6)) * 2; i0 < B; i0 += G * (NT / 64) * 2) {
        const int lane = tid & 31, i = i0 + ((tid >> 5) & 1);
        const int32_t y = i < B ? cands.label(i) : -1; // list position 0: the sample's own class, -1 if it is not one of this GPU's
        const bool own = y >= 0 && y < C;
        const int word = own ? y >> 5 : 0, below = word & 31;
        uint32_t v = bm[(word & ~31) + lane];
        if (lane > below) v = 0u;
        if (lane == below) v &= (1u << (y & 31)) - 1u;
        int p = __popc(v);
        p += KS_DPP(0, p, 0x111, 0xf);
        p += KS_DPP(0, p, 0x112, 0xf);
        p += KS_DPP(0, p, 0x114, 0xf);
        p += KS_DPP(0, p, 0x118, 0xf);
        p += KS_DPP(0, p, 0x142, 0xa); // the last lane of each half has its half's sum
        if (lane == 31 && i < B) {
            p = own ? coarse[word >> 5] + p : none;
            target_pos[i] = (p >= 0 && p < n) ? p : none;
        }
    }
    if (g == 0 && tid == 0) {
        *n_active = n;
        if (n_found) *n_found = found;
    }
}


// The selection of the NEXT batch as extra workgroups of the step's launches (nsel == 0: none): `nfetch` blocks of
// `fetch_nt` threads stage the candidates (they ride along with the dX launch), `nsel` workgroups select (with the dW
// launch, which leaves compute units idle).  The candidates come from the dense graph of a GPU that owns all classes
// or from the compressed graph of one node (csr_source), then with that selection's fill-up if asked for.
struct KsSelNext {
    int nsel, nfetch;
    int csr_source;
    SelDense dense;
    SelCsr csr;
    SelPad pad;
    int64_t C; // classes the bitmap covers (all classes, or the node's)
    int B, K, M;
    int32_t *cand;
    int32_t *active_idx, *n_active, *n_found, *target_pos;
    int32_t *dev_status;
};
template <int NT> __device__ __forceinline__ void ks_sel_next_fetch(const KsSelNext &s, int block) {
    const int64_t t = (int64_t)block * NT + threadIdx.x;
    if (t >= (int64_t)s.B * (s.K + 1)) return;
    const int i = (int)(t / (s.K + 1)), r = (int)(t % (s.K + 1));
    s.cand[(int64_t)r * s.B + i] = s.csr_source ? s.csr.cand(i, r, s.dev_status) : s.dense.cand(i, r, s.dev_status);
}
template <int NT> __device__ __forceinline__ void ks_sel_next_select(const KsSelNext &s, uint32_t *lds, int g) {
    Sel1Staged<NT> cands{s.cand, s.B, s.K, nullptr};
    sel1_body<NT>(lds, cands, s.C, s.B, s.K, s.M, s.csr_source, s.pad, s.active_idx, s.n_active, s.n_found, s.target_pos,
                  s.nsel, g);
}
