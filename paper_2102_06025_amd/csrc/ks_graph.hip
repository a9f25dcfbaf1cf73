// Exact KNN graph of the class-weight rows (paper Section 3.2.2: linear search with inner-product
// similarity; 16-bit matrix-core pass that recalls k' > K candidates, then an exact re-rank).
//
//   prepare   bf16 copy of W when the input is fp32; row norms and their maximum (for the error bound); the sampled rows
//   threshold (K <= 64, D <= 512) per row the 8th, 10th or 12th largest similarity to a sample of one in 32 (or 16) of the searched rows: what lies below
//             it is not recalled.  Some 256 to 384 rows (one in 16: 128 to 192) lie above it, whatever the data (an order statistic).
//   recall    each workgroup keeps a block of 256 rows resident and streams rows of W by them: bf16 MFMA tiles of
//             similarities; an element above its row's threshold is appended to one of the row's candidate segments.
//             The C x C similarities are never stored.  Small problems cut the streamed rows into parts so that every
//             compute unit has work.  Large problems (D = 128, 256, 512) take the variant that computes every similarity
//             once and uses it for both rows of the pair (gr_sym_*).  K > 64 or D > 512: a running threshold per row
//             instead of the sample's (a full candidate buffer is cut back to its k' best).
//   rank      one wavefront per row: the candidates that can be among the K best by the error bound (a bitwise search for
//             the K-th key), their canonical fp64 similarities, exact order (similarity descending, id ascending), first K written out.  The row is
//             certified when the K-th exact similarity exceeds the largest dropped one by more than the error bound of
//             the matrix-core pass; otherwise it is ranked again over all its candidates, and failing that goes to
//   exhaustive  uncertified rows are searched over all C columns in canonical fp64 arithmetic.
// Every decision that reaches the output is taken on the canonical fp64 similarity, so the lists are
// exact and do not depend on scheduling.
#include "ks_gemm.h"
#include "ks_gemm_async.h"
#include "ks_gemm_soe.h"

typedef KsTile<128, 128, 64, 2, 2> TileR;       // generic recall tile (any D % 32 == 0)
typedef KsATile<256, 256, 2, 4, 2> TileRA;      // asynchronous recall tile (D % 64 == 0)

#define GR_NT 256
#define GR_FB_BLOCKS 64   /* workgroups (and fp64 scratch rows) of the exhaustive pass */
#define GR_MAX_D 4096     /* the exhaustive pass keeps one row in LDS as fp64 */

__device__ __forceinline__ uint32_t gr_orderable(float f) {
    const uint32_t u = __float_as_uint(f); // negative: all bits flipped; otherwise: the sign bit set
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float gr_unorder(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// The two sides of a recall pass: the rows whose neighbours are searched (resident in the workgroups) and the rows
// that are searched (streamed past them).  The graph build searches W in W; one hop of the distributed build
// searches the node's rows in a visiting shard.
struct GrPair {
    const uint16_t *R; // [Cr, D]
    int64_t Cr;
    const uint16_t *S; // [Cs, D]
    int64_t Cs;
    int64_t self;      // streamed row i + self is resident row i itself and is skipped
};

struct GrParams {
    int kprime; // candidates kept per row by the recall pass (48, 64, 128 or 256)
    int cap;    // candidate buffer entries per row (256 or 512)
};
// The recall pass keeps k' > K candidates so that the K-th exact similarity clears the recall threshold by more than
// the error bound of the 16-bit pass.  With fp32 rows that bound is dominated by their rounding to bf16 (0.4 % of
// |w_i||w_j|) and k' = 2 K gives the margin; with bf16 rows only the fp32 accumulation is left (D * 2^-23), orders
// of magnitude below the spacing of neighbouring similarities, and k' = 1.5 K is kept: the number of candidates a
// row collects during the sweep, and with it the epilogue's work, grows in proportion to k'.
static GrParams gr_params(int K, int D, int dtype = KS_DTYPE_FP32) {
    GrParams p;
    if (K <= 32) { p.kprime = dtype == KS_DTYPE_BF16 ? 48 : 64; p.cap = 256; }
    else if (K <= 64) { p.kprime = 128; p.cap = 256; }
    else { p.kprime = 256; p.cap = 512; }
    if (D % 64 == 0 && !(D == 128 || D == 256 || D == 512))
        p.cap = 512; // the 256 x 256 asynchronous recall kernel appends up to 256 candidates per row and tile
    return p;
}

// ------------------------------------------------------------------------------------------------
// prepare
// ------------------------------------------------------------------------------------------------
template <typename IN> struct GrElem;
template <> struct GrElem<uint16_t> {
    static __device__ __forceinline__ float f(uint16_t v) { return ks_bf2f(v); }
};
template <> struct GrElem<float> {
    static __device__ __forceinline__ float f(float v) { return v; }
};

// One pass over the rows of up to two matrices (a hop has two): norms in fp32 (only used for the error bound, with
// slack), their maximum per workgroup, the bf16 copy of fp32 rows, the copy of the sampled rows; and the counters of the
// later kernels are cleared.  HBM-bound.  A row is read by as many lanes as it has 16-byte pieces (a wavefront reads four
// rows of 128 bf16 at once), four row groups in flight per wavefront.  The maximum goes to memory once per workgroup: an
// atomic per row on one address serialised in the L2 (10,000 x 128 fp32: 53 us; 390,625 x 512 bf16: 232 us).
#define GR_PREP_BLOCKS 1024
struct GrPrepJob {
    const void *W;
    int64_t C;
    uint16_t *Wb;    // bf16 copy, or nullptr
    float *norms;    // [C], or nullptr
    float *blockmax; // largest norm seen by each of this job's workgroups
    uint16_t *Ws;    // [n_sample, D] rows picked by gr_sample_row, or nullptr
    int64_t n_sample;
    int every;       // rows per sampled row
    int blocks;
};
struct GrClear {
    int32_t *fb_count, *second_count, *logcnt;
    int nlog;
    float *thf; // thresholds of the padding rows [pad0, pad1): nothing passes
    int64_t pad0, pad1;
};
// rows sampled: one of every 32 (or 16) consecutive rows, at a position that varies from one run of rows to the next
__device__ __forceinline__ int64_t gr_sample_row(int64_t s, int every) { // every: a power of two
    return s * every + (int64_t)((((uint32_t)s * 2654435761u) >> 16) & (uint32_t)(every - 1));
}
template <typename IN>
__global__ void __launch_bounds__(GR_NT)
gr_prepare_kernel(GrPrepJob job0, GrPrepJob job1, int D, GrClear clr) {
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            *clr.fb_count = 0;
            if (clr.second_count) *clr.second_count = 0;
        }
        for (int q = threadIdx.x; q < clr.nlog; q += GR_NT) clr.logcnt[q] = 0;
        for (int64_t q = clr.pad0 + threadIdx.x; q < clr.pad1; q += GR_NT) clr.thf[q] = INFINITY;
    }
    const bool second = (int)blockIdx.x >= job0.blocks;
    const GrPrepJob job = second ? job1 : job0;
    const int bid = second ? (int)blockIdx.x - job0.blocks : (int)blockIdx.x;
    constexpr int EPL = 16 / sizeof(IN), U = 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int lpr = 64; // lanes per row
    while (lpr > 4 && (lpr >> 1) * EPL >= D) lpr >>= 1;
    const int l = lane & (lpr - 1), rpw = 64 / lpr;
    const int64_t stride = (int64_t)job.blocks * (GR_NT / 64) * rpw;
    const IN *__restrict__ W = (const IN *)job.W;
    const int every_log = job.Ws ? __builtin_ctz(job.every) : 0;
    float mx = 0.f;
    for (int64_t i0 = ((int64_t)bid * (GR_NT / 64) + wave) * rpw + lane / lpr; i0 < job.C; i0 += U * stride) {
        float s[U];
        bool pick[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u * stride;
            s[u] = 0.f;
            const int64_t sm = i >> every_log;
            pick[u] = job.Ws && sm < job.n_sample && gr_sample_row(sm, job.every) == i;
        }
        for (int d = l * EPL; d < D; d += lpr * EPL) {
            uint4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = i0 + u * stride;
                v[u] = i < job.C ? *(const uint4 *)(W + i * D + d) : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = i0 + u * stride;
                if (i >= job.C) continue;
                const uint32_t w4[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                if (sizeof(IN) == 2) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float lo = __uint_as_float(w4[e] << 16), hi = __uint_as_float(w4[e] & 0xFFFF0000u);
                        s[u] = fmaf(lo, lo, s[u]);
                        s[u] = fmaf(hi, hi, s[u]);
                    }
                    if (pick[u]) *(uint4 *)(job.Ws + (i >> every_log) * D + d) = v[u];
                } else {
                    float f[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        f[e] = __uint_as_float(w4[e]);
                        s[u] = fmaf(f[e], f[e], s[u]);
                    }
                    const uint2 b = make_uint2(ks_pack_bf2(f[0], f[1]), ks_pack_bf2(f[2], f[3]));
                    *(uint2 *)(job.Wb + i * D + d) = b;
                    if (pick[u]) *(uint2 *)(job.Ws + (i >> every_log) * D + d) = b;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u * stride;
            for (int o = 1; o < lpr; o <<= 1) s[u] += __shfl_xor(s[u], o, 64);
            const float nrm = sqrtf(s[u]);
            mx = fmaxf(mx, nrm);
            if (i < job.C && l == 0 && job.norms) job.norms[i] = nrm;
        }
    }
    __shared__ float s_mx[GR_NT / 64];
    mx = ks_wave_max(mx);
    if (lane == 0) s_mx[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < GR_NT / 64; ++w) mx = fmaxf(mx, s_mx[w]);
        job.blockmax[bid] = mx;
    }
}
// largest row norm from the workgroups' maxima; every lane of a wavefront gets it
__device__ __forceinline__ float gr_max_norm(const float *__restrict__ blockmax, int n) {
    float mx = 0.f;
    for (int q = threadIdx.x & 63; q < n; q += 64) mx = fmaxf(mx, blockmax[q]);
    return ks_wave_max(mx);
}
__global__ void __launch_bounds__(64) gr_maxnorm_kernel(const float *__restrict__ blockmax, int n, float *maxnorm) {
    const float mx = gr_max_norm(blockmax, n);
    if (threadIdx.x == 0) *maxnorm = mx;
}

// Cut the candidate buffer of one row back to its kprime best (in no particular order: the exact stage ranks them
// anyway) and make the kprime-th best value the row's new threshold; updates cnt/thr in LDS.  One wavefront per row.
// The kprime-th largest key is found by a bitwise search -- rounds of "how many keys are >= this prefix", each a
// compare per key, a wavefront ballot and a population count -- which is an order of magnitude cheaper than sorting
// the keys across the lanes (the keys are distinct: value bits above, inverted row id below; empty slots are 0).
// The 32 value bits are searched first; the id bits only when several keys share the kprime-th value.
// Requires kprime <= number of keys.
template <int E> __device__ __forceinline__ int gr_count_hi_ge(const uint64_t (&val)[E], uint32_t t) {
    int c = 0;
#pragma unroll
    for (int r = 0; r < E; ++r) c += __popcll(__ballot((uint32_t)(val[r] >> 32) >= t));
    return c;
}
template <int E> __device__ __forceinline__ int gr_count_lo_ge(const uint64_t (&val)[E], uint32_t hi, uint32_t t) {
    int c = 0;
#pragma unroll
    for (int r = 0; r < E; ++r) c += __popcll(__ballot((uint32_t)(val[r] >> 32) == hi && (uint32_t)val[r] >= t));
    return c;
}
template <int E>
__device__ __forceinline__ void gr_compact_row(uint64_t *__restrict__ cand_row, int *cnt, uint32_t *thr, int kprime) {
    const int lane = threadIdx.x & 63;
    const int n = *cnt;
    uint64_t val[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        int idx = r * 64 + lane;
        val[r] = idx < n ? cand_row[idx] : 0ull; // 0 is below every real key
    }
    uint32_t t_hi = 0; // every decision below is uniform over the wavefront
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t c = t_hi | (1u << bit);
        if (gr_count_hi_ge<E>(val, c) >= kprime) t_hi = c;
    }
    uint64_t t = (uint64_t)t_hi << 32;
    if (gr_count_hi_ge<E>(val, t_hi) != kprime) { // keys of equal value straddle the cut: the ids decide
        const int need = kprime - (t_hi == 0xFFFFFFFFu ? 0 : gr_count_hi_ge<E>(val, t_hi + 1u));
        uint32_t t_lo = 0;
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t c = t_lo | (1u << bit);
            if (gr_count_lo_ge<E>(val, t_hi, c) >= need) t_lo = c;
        }
        t |= t_lo;
    }
    // t is the kprime-th largest key: exactly kprime keys are >= t; they move to the front of the buffer
    int base = 0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint64_t m = __ballot(val[r] >= t);
        if (val[r] >= t) cand_row[base + __popcll(m & ((1ull << lane) - 1ull))] = val[r];
        base += __popcll(m);
    }
    if (lane == 0) {
        *cnt = kprime;
        *thr = (uint32_t)(t >> 32);
    }
}

// ------------------------------------------------------------------------------------------------
// recall pass
// ------------------------------------------------------------------------------------------------
template <class T, int E>
__global__ void __launch_bounds__(T::NT)
gr_recall_kernel(GrPair pr, int D, int kprime, uint64_t *__restrict__ cand, int32_t *__restrict__ cnt_out,
                 uint32_t *__restrict__ thr_out) {
    const int64_t C = pr.Cr;
    constexpr int CAP = E * 64;
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::LDS_ELEMS];
    __shared__ int s_cnt[T::BM];
    __shared__ uint32_t s_thr[T::BM];
    const int wave = threadIdx.x >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * T::BM;
    for (int m = threadIdx.x; m < T::BM; m += T::NT) { s_cnt[m] = 0; s_thr[m] = 0u; }
    __syncthreads();

    KsRowLoader<T::BM, T::BK, T::NT> al;
    al.init(pr.R, D, nullptr, (int)row0, (int)C, D);
    const int n_col_blocks = (int)((pr.Cs + T::BN - 1) / T::BN);
    const int nk = (D + T::BK - 1) / T::BK;
    for (int J = 0; J < n_col_blocks; ++J) {
        KsRowLoader<T::BN, T::BK, T::NT> bl;
        bl.init(pr.S, D, nullptr, J * T::BN, (int)pr.Cs, D);
        f32x16_t acc[T::FM][T::FN];
        ks_tile_clear<T>(acc);
        ks_gemm_mainloop<T>(al, bl, 0, nk, lds, acc);
        ks_tile_foreach<T>(acc, [&](int m, int n, float v) {
            const int64_t i = row0 + m, j = (int64_t)J * T::BN + n;
            if (i < C && j < pr.Cs && j != i + pr.self) {
                const uint32_t hi = gr_orderable(v);
                if (hi > s_thr[m]) {
                    int slot = atomicAdd(&s_cnt[m], 1);
                    if (slot < CAP) // always true: a buffer is cut back before it can overflow
                        cand[i * CAP + slot] = ((uint64_t)hi << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)j);
                }
            }
        });
        __syncthreads();
        for (int m = wave; m < T::BM; m += T::NT / 64) {
            if (s_cnt[m] > CAP - T::BN) gr_compact_row<E>(cand + (row0 + m) * CAP, &s_cnt[m], &s_thr[m], kprime);
        }
        __syncthreads();
    }
    for (int m = wave; m < T::BM; m += T::NT / 64) {
        if (row0 + m < C) {
            if (s_cnt[m] > kprime) gr_compact_row<E>(cand + (row0 + m) * CAP, &s_cnt[m], &s_thr[m], kprime);
        }
    }
    __syncthreads();
    for (int m = threadIdx.x; m < T::BM; m += T::NT) {
        if (row0 + m < C) { cnt_out[row0 + m] = s_cnt[m]; thr_out[row0 + m] = s_thr[m]; }
    }
}

// ------------------------------------------------------------------------------------------------
// recall pass on the asynchronous engine (D % 64 == 0): 256 rows per workgroup, 256-column blocks.
// The k-tiles of the whole sweep form one stream: the first k-tile of the next column block is already
// on its way into LDS while the current block's similarities are filtered.
// ------------------------------------------------------------------------------------------------
template <class T, int E>
__global__ void __launch_bounds__(T::NT)
gr_recall_async_kernel(GrPair pr, int D, int kprime, uint64_t *__restrict__ cand, int32_t *__restrict__ cnt_out,
                       uint32_t *__restrict__ thr_out) {
    const int64_t C = pr.Cr;
    constexpr int CAP = E * 64;
    static_assert(T::STAGES == 2 && CAP >= 256 + T::BN, "recall tile");
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::LDS_ELEMS];
    __shared__ int s_cnt[T::BM];
    __shared__ uint32_t s_thr[T::BM];
    const int wave = threadIdx.x >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * T::BM;
    for (int m = threadIdx.x; m < T::BM; m += T::NT) { s_cnt[m] = 0; s_thr[m] = 0u; }
    __syncthreads();

    KsARows<T::BM, T::NW> ar;
    KsARows<T::BN, T::NW> br;
    ar.init(pr.R, D, nullptr, (int)row0, (int)C);
    br.init(pr.S, D, nullptr, 0, (int)pr.Cs);
    const int nJ = (int)((pr.Cs + T::BN - 1) / T::BN), nk = D / 64;
    // stream position of the next tile to load
    int ld_J = 0, ld_kt = 0;
    auto issue_next = [&](int stage) {
        uint16_t *st = lds + stage * T::STAGE_ELEMS;
        ar.issue(ld_kt * 64, st);
        br.issue(ld_kt * 64, st + T::BM * 64);
        if (++ld_kt == nk) {
            ld_kt = 0;
            ++ld_J;
            if (ld_J < nJ) br.init(pr.S, D, nullptr, ld_J * T::BN, (int)pr.Cs);
        }
    };
    issue_next(0);
    int stage = 0;
    for (int J = 0; J < nJ; ++J) {
        f32x16_t acc[T::FM][T::FN];
        ks_a_clear<T>(acc);
        for (int kt = 0; kt < nk; ++kt) {
            ks_wait_vmcnt<0>();
            ks_barrier_nofence();
            if (ld_J < nJ) issue_next(stage ^ 1);
            ks_a_tile_mma<T>(lds + stage * T::STAGE_ELEMS, acc);
            stage ^= 1;
        }
        ks_a_foreach<T>(acc, [&](int m, int n, float v) {
            const int64_t i = row0 + m, j = (int64_t)J * T::BN + n;
            if (i < C && j < pr.Cs && j != i + pr.self) {
                const uint32_t hi = gr_orderable(v);
                if (hi > s_thr[m]) {
                    int slot = atomicAdd(&s_cnt[m], 1);
                    if (slot < CAP) // always true: a buffer is cut back before it can overflow
                        cand[i * CAP + slot] = ((uint64_t)hi << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)j);
                }
            }
        });
        __syncthreads();
        for (int m = wave; m < T::BM; m += T::NW) {
            if (s_cnt[m] > CAP - T::BN) gr_compact_row<E>(cand + (row0 + m) * CAP, &s_cnt[m], &s_thr[m], kprime);
        }
        __syncthreads();
    }
    for (int m = wave; m < T::BM; m += T::NW) {
        if (row0 + m < C) {
            if (s_cnt[m] > kprime) gr_compact_row<E>(cand + (row0 + m) * CAP, &s_cnt[m], &s_thr[m], kprime);
        }
    }
    __syncthreads();
    for (int m = threadIdx.x; m < T::BM; m += T::NT) {
        if (row0 + m < C) { cnt_out[row0 + m] = s_cnt[m]; thr_out[row0 + m] = s_thr[m]; }
    }
}

// ------------------------------------------------------------------------------------------------
// recall pass as a stationary-operand sweep (D = 128, 256 or 512): a workgroup keeps the MFMA fragments
// of its 256 rows in registers and streams every row of W past them, 96 rows at a time.  A lane owns one
// of the 256 rows in the accumulators, so the row's threshold is a register and most elements cost one
// max operation; only groups of four elements whose maximum beats the threshold are looked at one by one.
// ------------------------------------------------------------------------------------------------
#define GR_SOE_STAGES 6
// Candidate buffers of the sweep kernel below.  Two lanes of a wavefront share a row of the graph (they hold
// different streamed rows of it), so each appends to its own half of the row's buffer and counts in a register:
// an append is a store and an increment, with no atomic operation and nothing to wait for.
// Cuts the two halves (n0 and n1 keys) back to the kprime largest keys and returns the value bits of the smallest
// key kept (0 when nothing was dropped); survivors go half and half to the two halves, or -- for the final call --
// to the front of the buffer.  One wavefront per row.
template <int E>
__device__ __forceinline__ uint32_t gr_compact_halves(uint64_t *__restrict__ cand_row, int n0, int n1, int kprime,
                                                       bool final_layout, int *n_kept) {
    constexpr int HALF = E * 32;
    const int lane = threadIdx.x & 63;
    uint64_t val[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = r * 64 + lane;
        const bool valid = idx < HALF ? idx < n0 : idx - HALF < n1;
        val[r] = valid ? cand_row[idx] : 0ull; // 0 is below every real key
    }
    const int n = n0 + n1;
    uint64_t t = 1ull; // keeps every real key
    if (n > kprime) {
        uint32_t t_hi = 0; // every decision below is uniform over the wavefront
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t c = t_hi | (1u << bit);
            if (gr_count_hi_ge<E>(val, c) >= kprime) t_hi = c;
        }
        t = (uint64_t)t_hi << 32;
        if (gr_count_hi_ge<E>(val, t_hi) != kprime) { // keys of equal value straddle the cut: the ids decide
            const int need = kprime - (t_hi == 0xFFFFFFFFu ? 0 : gr_count_hi_ge<E>(val, t_hi + 1u));
            uint32_t t_lo = 0;
            for (int bit = 31; bit >= 0; --bit) {
                const uint32_t c = t_lo | (1u << bit);
                if (gr_count_lo_ge<E>(val, t_hi, c) >= need) t_lo = c;
            }
            t |= t_lo;
        }
    }
    const int kept = n > kprime ? kprime : n;
    const int first = final_layout ? kept : (kept + 1) / 2; // keys that go to the first half
    int base = 0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint64_t m = __ballot(val[r] >= t);
        if (val[r] >= t) {
            const int q = base + __popcll(m & ((1ull << lane) - 1ull));
            cand_row[q < first ? q : HALF + (q - first)] = val[r];
        }
        base += __popcll(m);
    }
    *n_kept = kept;
    return n > kprime ? (uint32_t)(t >> 32) : 0u;
}

template <int KT, int E>
__global__ void __launch_bounds__(512)
gr_recall_soe_kernel(GrPair pr, int D, int kprime, uint64_t *__restrict__ cand, int32_t *__restrict__ cnt_out,
                      uint32_t *thr_out, const uint32_t *thr_init) {
    const int64_t C = pr.Cr;
    typedef KsSoe<KT, 96, GR_SOE_STAGES, 2> CFG;
    constexpr int CAP = E * 64, HALF = CAP / 2;
    constexpr int LIMIT = HALF - CFG::FM * 16; // a lane appends at most FM * 16 keys per chunk
    static_assert(LIMIT >= 64, "room for half of the largest kprime of this buffer size");
    __shared__ __attribute__((aligned(16))) uint16_t lds[CFG::LDS_ELEMS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * CFG::RES;
    const int col = ks_soe_col();
    const int gi = (int)row0 + col; // C < 2^31
    const int Ci = (int)C;
    const int64_t self0 = row0 + pr.self; // streamed rows [self0, self0 + RES) are this workgroup's own rows
    // A wavefront's accumulators hold 32 of the 256 rows, two lanes per row (lane and lane + 32 hold different streamed
    // rows), so the candidate buffers of those rows are written by that wavefront alone: it also cuts them back
    // itself, the counts and the thresholds live in registers, and the epilogue needs no barrier and no atomics.
    // an append is a store at a 32-bit slot number behind one base address of the workgroup: the count of the lane's
    // half plus a constant of the lane
    uint64_t *const wg_cand = cand + row0 * CAP;
    const uint32_t my_base = (uint32_t)(col * CAP + (lane >> 5) * HALF);
    int my_cnt = 0;
    uint32_t th = 0u; // value bits of the row's threshold; 0 = nothing dropped yet: everything passes
    float thf = gi >= Ci ? INFINITY : -INFINITY; // rows beyond C never pass
    if (thr_init && gi < Ci) { // the caller knows that nothing at or below this value is wanted (may be thr_out itself)
        th = thr_init[gi];
        if (th != 0u) thf = gr_unorder(th);
    }
    auto cut_back = [&](bool final_layout) {
        ks_wait_vmcnt<0>(); // the appended candidates have left this wavefront before it reads them back
        asm volatile("" ::: "memory");
        for (int m = 0; m < 32; ++m) {
            const int n0 = __builtin_amdgcn_readlane(my_cnt, m), n1 = __builtin_amdgcn_readlane(my_cnt, m + 32);
            if (final_layout ? (row0 + wave * 32 + m < C) : (n0 > LIMIT || n1 > LIMIT)) {
                int kept;
                const uint32_t t = gr_compact_halves<E>(cand + (row0 + wave * 32 + m) * CAP, n0, n1, kprime, final_layout, &kept);
                if ((lane & 31) == m) {
                    my_cnt = final_layout ? kept : (lane < 32 ? (kept + 1) / 2 : kept / 2);
                    if (t != 0u) { th = t; thf = gr_unorder(t); }
                }
            }
        }
        asm volatile("" ::: "memory");
    };
    auto epi = [&](int c0, int rows_here, f32x16_t (&acc)[CFG::FM]) {
        // elements that need more than the threshold test: the tail of the last chunk, and the diagonal
        const bool special = rows_here < CFG::CH || ((int64_t)c0 < self0 + CFG::RES && (int64_t)c0 + CFG::CH > self0);
        constexpr int GROUP = 4; // elements per threshold test (2 .. 16 measured alike)
        // compiled twice: nearly all chunks are plain (all rows real, none of them the row itself)
        auto elements = [&](auto is_special) __attribute__((always_inline)) {
            constexpr bool SPECIAL = decltype(is_special)::value;
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm) {
#pragma unroll
                for (int q = 0; q < 16 / GROUP; ++q) { // GROUP elements at a time: most groups have none that passes
                    float bm = acc[fm][q * GROUP];
#pragma unroll
                    for (int e = 1; e < GROUP; ++e) bm = fmaxf(bm, acc[fm][q * GROUP + e]);
                    if (bm > thf) {
#pragma unroll
                        for (int e = 0; e < GROUP; ++e) {
                            const int r = q * GROUP + e;
                            const float v = acc[fm][r];
                            if (v > thf) {
                                const int lr = ks_soe_row(fm, r, lane);
                                const int j = c0 + lr;
                                if (SPECIAL && (lr >= rows_here || (int64_t)j == (int64_t)gi + pr.self)) continue;
                                // (my_cnt < HALF: a buffer is cut back before it can overflow; the mask keeps the
                                // store inside the lane's half whatever happens)
                                wg_cand[my_base + ((uint32_t)my_cnt & (uint32_t)(HALF - 1))] =
                                    ((uint64_t)gr_orderable(v) << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)j);
                                ++my_cnt;
                            }
                        }
                    }
                }
            }
        };
        if (special) elements(std::true_type());
        else elements(std::false_type());
        if (__any(my_cnt > LIMIT)) cut_back(false); // a buffer could overflow in the next chunk
    };
    ks_soe_sweep<CFG>(pr.R, D, (int)row0, (int)C, pr.S, D, nullptr, 0, (int)pr.Cs, (int)pr.Cs, lds, epi);
    cut_back(true); // at most kprime keys per row, at the front of its buffer
    if (lane < 32 && gi < Ci) { cnt_out[gi] = my_cnt; thr_out[gi] = th; }
}

// ------------------------------------------------------------------------------------------------
// Recall with thresholds fixed beforehand (K <= 64, D <= 512).
//
// A first sweep (gr_threshold_kernel) finds for every row its r-th largest similarity to a sample of one in 32 of the
// searched rows; r = 8 for K <= 16, 10 for K <= 32, 12 for K <= 64.  The number of searched rows at or above it is
// 32 * Gamma(r) whatever their distribution (an order statistic of a uniform sample): 256, 320 or 384 on average.
// (Smaller builds: one in 16, see gr_every.)  The
// largest K of each r is the worst case: beyond 1,152, 1,280 and 1,408 (what a row's segments take, see GrSegs) for less than
// five rows in a billion; at most K (then r of the row's K + 1 best would have to be in the sample) for 0.1 to 1.4 in a
// million, and for 1.0, 1.1 and 8.3 in a million of the rows that are in their own sample.
// The candidate segments are sized for those counts and nothing is cut back during the sweep, so that
//   * a row's candidates may come from several workgroups: gr_recall_fix_kernel cuts the searched rows into `parts`, one
//     workgroup per (256 resident rows, part).  10,000 rows are 40 blocks; with one workgroup each, 216 compute units idle.
//   * a similarity may serve both of its rows: gr_recall_sym_kernel.
// A row that does end up with too many or too few candidates is caught by the certificate like any other uncertain row.
// ------------------------------------------------------------------------------------------------
#define GR_SYM_Q 512             /* symmetric sweep: slots of a candidate segment (one lane's hits) */
#define GR_SYM_SCAP 1024         /* slots of the stream-side segment */
#define GR_MAX_CAND 2048         /* candidates of a row that the ranking takes */
#define GR_RANK 12               /* places of the sorted list that finds a row's threshold */
#define GR_SAMPLE_PARTS 8        /* workgroups per block of resident rows that search the sample, at most */
#define GR_MAX_PARTS 24
#define GR_CUS 256               /* compute units that the parts are planned for */

// A row's candidate segments: 2 * parts of q slots (the two lanes of a part that hold the row), then `stream` slots.
// Symmetric sweep: a lane has its q slots.  Passes with parts (no stream segment): the two lanes of a part share 2 q slots and
// fill them from both ends, so that however a row's hits fall on lanes and parts, all of them fit: a lane sees the streamed
// rows whose id has bit 2 clear, or set, and neighbours with ids of one residue modulo 8 are all one lane's.  2 q = 64 (r + 10),
// and what a lane can find in one chunk of 96 rows, before which it looks whether it has room (in turns: in a block of 32).
// (With 512 slots for each lane, four rows in 100,000 of K > 32 overflowed even with hits that fall evenly, and a row in the
// exhaustive search costs 4 to 30 ms: 60,000 x 128, K = 64: 5.6 ms instead of 2.0; a hop of 65,000 rows of 512 against
// a million 194 ms instead of 57.)
struct GrSegs {
    int parts, q, stream;
    __host__ __device__ int cap() const { return 2 * parts * q + stream; }
};
// What is in the segments of a row: lane s gets the count of segment s (0 beyond the last) and where it begins.  Returns
// whether one has overflowed, which makes all counts 0.  All lanes of a wavefront call.
__device__ __forceinline__ bool gr_segments(const GrSegs &seg, const int32_t *__restrict__ cnt_res, const int32_t *__restrict__ cnt_str,
                                            int64_t i, int &c, int &begin) {
    const int lane = threadIdx.x & 63, nres = 2 * seg.parts;
    int most = seg.q;
    c = 0;
    if (lane < nres) c = cnt_res[i * nres + lane];
    else if (lane == nres && seg.stream > 0) { c = cnt_str[i]; most = seg.stream; }
    begin = lane * seg.q;
    if (seg.stream == 0) {
        most = 2 * seg.q - KS_DPP(0, c, 0xB1, 0xf); // what the other lane of the pair has left
        if (lane & 1) begin += seg.q - c;           // from the end downwards
    }
    const bool overflow = __ballot(c > most) != 0ull;
    if (overflow) c = 0;
    return overflow;
}
// Shape of the sweeps (ks_soe_pp_sweep) for a depth of KT k-tiles: as many rows per chunk as two sets of accumulators beside the resident fragments
// allow, and as few stages per chunk as the LDS allows with three in flight: a stage is a barrier, at which the wavefront with
// the most hits keeps the others waiting.  (100,000 x 256: one stage per chunk 4.40 ms, two 4.51, four 4.77; 100,000 x 128:
// one 3.76, two 3.81; 390,625 x 512: two 81.0 ms, four 82.9.)  Whole builds, plain sweep -> in turns: 390,625 x 512, K = 32: 82.8 ->
// 80.1 ms; 300,000 x 128: 26.1 -> 22.7; 200,000 x 256: 19.5 -> 17.2; 100,000 x 256: 5.01 -> 4.32; 60,000 x 320: 2.89 -> 2.58; 70,000 x 192:
// 2.97 -> 2.48; 40,000 x 448: 1.73 -> 1.57; 20,000 x 96: 257 -> 242 us; 10,000 x 128 fp32: 123 -> 118.  (The pass over every similarity once
// spills 6 registers at KT = 8 and 16 at KT = 2; smaller chunks or fewer k-steps ahead spill nothing and are slower: 150,000 x 128 7.51 ->
// 7.76 ms, 390,625 x 512 80.1 -> 80.6.)
template <int KT, bool RAGGED> struct GrPpOf;
#define GR_PP(KT, ...) \
    template <bool RAGGED> struct GrPpOf<KT, RAGGED> { typedef KsPp<KT, __VA_ARGS__, RAGGED> T; };
GR_PP(1, 4, 1, 5, 2)
GR_PP(2, 4, 2, 4, 2)
GR_PP(3, 3, 3, 4, 2)
GR_PP(4, 3, 4, 3, 2)
GR_PP(5, 2, 5, 3, 4)
GR_PP(6, 2, 6, 3, 2)
GR_PP(7, 1, 7, 4, 4)
GR_PP(8, 2, 4, 4, 3)
#undef GR_PP
template <int KT, bool RAGGED> using GrPp = typename GrPpOf<KT, RAGGED>::T;
// The thresholds' sorted lists take 24 registers more, hence chunks of 32 or 64 rows.  gr_threshold_kernel, plain, in turns (on one card,
// us): 150,000 x 64 409, 416; x 96 435, 438; x 128 522, 521; x 192 570, 557; x 256 676, 608; 100,000 x 320 347, 333; x 384 367, 353; x 448
// 417, 403; x 512 453, 428; 390,625 x 512 4,995, 4,822.  Small problems (several workgroups per block of rows) have a chunk or two per
// workgroup, with nothing to take turns in, and stay on the plain sweep (10,000 x 128: 11.6 us, in turns 17).
template <int KT, bool RAGGED> struct GrThrPpOf;
#define GR_THR_PP(KT, ...) \
    template <bool RAGGED> struct GrThrPpOf<KT, RAGGED> { typedef KsPp<KT, __VA_ARGS__, RAGGED> T; };
GR_THR_PP(1, 2, 1, 8, 2)
GR_THR_PP(2, 2, 2, 5, 2)
GR_THR_PP(3, 2, 3, 3, 2)
GR_THR_PP(4, 2, 4, 3, 2)
GR_THR_PP(5, 2, 5, 3, 2)
GR_THR_PP(6, 2, 6, 3, 2)
GR_THR_PP(7, 1, 7, 4, 4)
GR_THR_PP(8, 1, 4, 8, 4)
#undef GR_THR_PP
template <int KT, bool RAGGED> using GrThrPp = typename GrThrPpOf<KT, RAGGED>::T;
// Stage shape of the plain sweep: twelve k-tiles in flight, two per stage where KT is even (a barrier per stage); a single k-tile per
// chunk (KT = 1): six, which leaves LDS for a second workgroup.
template <int KT, bool RAGGED> using GrSoe = KsSoe<KT, 96, (KT % 2 == 0 || KT == 1) ? 6 : 12, KT % 2 == 0 ? 2 : 1, RAGGED>;
static int gr_chunk(int D) { // streamed rows per chunk of the recall passes
    switch ((D + 63) / 64) {
    case 1: return GrPp<1, false>::CH;
    case 2: return GrPp<2, false>::CH;
    case 3: return GrPp<3, false>::CH;
    case 4: return GrPp<4, false>::CH;
    case 5: return GrPp<5, false>::CH;
    case 6: return GrPp<6, false>::CH;
    case 7: return GrPp<7, false>::CH;
    default: return GrPp<8, false>::CH;
    }
}

// One hop of the distributed build: a row whose list is full needs no visiting row whose similarity cannot reach the
// list's last entry: its threshold is at least that entry's similarity, lowered by more than twice the recall's error
// bound (a visiting row that ties the entry exactly is still recalled, and the certificate of the merge -- new K-th
// similarity above threshold + bound -- holds when nothing new comes in).  graph == nullptr: no lists.
struct GrHop {
    const int32_t *graph;
    const double *sims;
    const float *norms;
    int K;
    float gamma;
};
__device__ __forceinline__ uint32_t gr_hop_threshold(const GrHop &hop, int64_t i, float maxnorm) {
    if (!hop.graph || hop.graph[i * hop.K + hop.K - 1] < 0) return 0u;
    const double eps = (double)hop.gamma * (double)hop.norms[i] * (double)maxnorm;
    const double want = hop.sims[i * hop.K + hop.K - 1] - 2.5 * eps;
    float f = (float)want;
    if ((double)f > want) f = nextafterf(f, -INFINITY); // rounded down
    return (f == f && f > -INFINITY) ? gr_orderable(f) : 0u;
}

// The r-th largest of the sorted lists of the two lanes that hold one row.  (Of a pair of places k, RANK - 1 - k the larger
// value is one of the RANK largest of both; what is left is sorted by inserting it again.)
__device__ __forceinline__ void gr_insert(float (&top)[GR_RANK], float v) { // top: descending
#pragma unroll
    for (int k = GR_RANK - 1; k > 0; --k) top[k] = __builtin_amdgcn_fmed3f(top[k - 1], top[k], v);
    top[0] = fmaxf(top[0], v);
}
__device__ __forceinline__ void gr_merge_halves(float (&top)[GR_RANK]) {
    float u[GR_RANK];
#pragma unroll
    for (int k = 0; k < GR_RANK; ++k) u[k] = -INFINITY;
#pragma unroll
    for (int k = 0; k < GR_RANK; ++k) gr_insert(u, fmaxf(top[k], __shfl_xor(top[GR_RANK - 1 - k], 32, 64)));
#pragma unroll
    for (int k = 0; k < GR_RANK; ++k) top[k] = u[k];
}
// Threshold of row i as a key (as a float: gr_unorder of it) from the descending list of its largest similarities to the
// sample: the float below the r-th largest, so that one passes.  "Key value <= threshold" holds for everything that fails.
__device__ __forceinline__ uint32_t gr_threshold_of(const float (&top)[GR_RANK], int r, const GrHop &hop, int64_t i, float maxnorm) {
    float t = -INFINITY;
#pragma unroll
    for (int k = 0; k < GR_RANK; ++k) t = k + 1 == r ? top[k] : t;
    const uint32_t lowest = gr_orderable(-INFINITY), tb = gr_orderable(t);
    const uint32_t bits = tb > lowest + 1u ? tb - 1u : lowest, hb = gr_hop_threshold(hop, i, maxnorm);
    return hb > bits ? hb : bits;
}
// How a sample is searched: rank of the threshold, workgroups per block of resident rows, sampled rows of each.  With one, the
// thresholds are ready when the kernel ends; with several, each leaves its sorted lists and the recall pass merges them
// (gr_merge_parts): 10,000 rows are 40 blocks, and the chip has 256 compute units.
struct GrSample {
    int r, parts, part_rows;
    float *tops; // [parts][GR_RANK][Cr], parts > 1
};

// A lane keeps the GR_RANK largest similarities of its row that it has seen, sorted, in registers: an insertion is one
// median-of-three per place.  (The first version appended to candidate buffers in memory and cut them back: every cut is
// 32 rows in turn per wavefront, 199 us for 10,000 rows of 128 against a sample of 312.)
// PARTS: whether smp.parts > 1.
template <int KT, bool RAGGED, bool PARTS>
__global__ void __launch_bounds__(512)
gr_threshold_kernel(const uint16_t *__restrict__ R, int64_t Cr, const uint16_t *__restrict__ Ws, int n_sample, int D,
                    GrSample smp, const float *__restrict__ blockmax, int n_blockmax, float *maxnorm, GrHop hop, float *__restrict__ thf,
                    uint32_t *__restrict__ tbits) {
    typedef typename std::conditional<PARTS, GrSoe<KT, RAGGED>, GrThrPp<KT, RAGGED>>::type CFG;
    __shared__ __attribute__((aligned(16))) uint16_t lds[CFG::LDS_ELEMS];
    const int id = PARTS ? ks_xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x, nb = PARTS ? gridDim.x / smp.parts : gridDim.x;
    const int part = PARTS ? id / nb : 0;
    const int64_t row0 = (int64_t)(PARTS ? id % nb : id) * CFG::RES;
    const int s0 = PARTS ? part * smp.part_rows : 0, s1 = PARTS && s0 + smp.part_rows < n_sample ? s0 + smp.part_rows : n_sample;
    float top[GR_RANK]; // descending
#pragma unroll
    for (int k = 0; k < GR_RANK; ++k) top[k] = -INFINITY;
    auto epi = [&](auto block, int, int rows_here, const f32x16_t &acc) __attribute__((always_inline)) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[4 * q + e];
            if (rows_here < CFG::CH) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (ks_soe_row(decltype(block)::value, 4 * q + e, lane) >= rows_here) v[e] = -INFINITY;
            }
            if (fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])) > top[GR_RANK - 1]) {
#pragma unroll
                for (int e = 0; e < 4; ++e) gr_insert(top, v[e]);
            }
        }
    };
    if constexpr (PARTS) {
        auto chunk = ks_soe_blocks<CFG>(epi);
        ks_soe_sweep<CFG>(R, D, (int)row0, (int)Cr, Ws, D, nullptr, s0, s1, n_sample, lds, chunk);
    } else {
        ks_soe_pp_sweep<CFG>(R, D, (int)row0, (int)Cr, Ws, D, s0, s1, n_sample, lds, epi);
    }
    gr_merge_halves(top); // the two lanes of a row hold disjoint sampled rows
    const float mx = (!PARTS && hop.graph) || id == 0 ? gr_max_norm(blockmax, n_blockmax) : 0.f;
    if (id == 0 && threadIdx.x == 0) *maxnorm = mx;
    const int64_t i = row0 + ks_soe_col();
    if ((threadIdx.x & 63) < 32 && i < Cr) {
        if (PARTS) {
#pragma unroll
            for (int k = 0; k < GR_RANK; ++k) smp.tops[((int64_t)part * GR_RANK + k) * Cr + i] = top[k];
        } else {
            const uint32_t bits = gr_threshold_of(top, smp.r, hop, i, mx);
            thf[i] = gr_unorder(bits);
            tbits[i] = bits;
        }
    }
}
// What the recall pass needs to merge the parts' lists, or nothing where the thresholds are ready.  (Two kernels: the merge as
// a branch of one made that one 1.5 % slower at every size that does not take it, 60,000 x 320: 2,486 -> 2,524 us.)
struct GrReady {};
struct GrMerge {
    GrSample smp;
    GrHop hop;
    const float *maxnorm;
    uint32_t *tbits; // for the ranking
};
// The threshold of row i (the same row in lanes l and l + 32) from the parts' lists; all lanes of a wavefront call.
__device__ __forceinline__ uint32_t gr_merge_parts(const GrMerge &merge, int64_t Cr, int64_t i) {
    const GrSample &smp = merge.smp;
    float top[GR_RANK];
#pragma unroll
    for (int k = 0; k < GR_RANK; ++k) top[k] = -INFINITY;
    const int64_t row = i < Cr ? i : Cr - 1;
    for (int p = (threadIdx.x >> 5) & 1; p < smp.parts; p += 2) { // the two lanes take every other part
        float v[GR_RANK];
#pragma unroll
        for (int k = 0; k < GR_RANK; ++k) v[k] = smp.tops[((int64_t)p * GR_RANK + k) * Cr + row];
#pragma unroll
        for (int k = 0; k < GR_RANK; ++k) gr_insert(top, v[k]);
    }
    gr_merge_halves(top);
    return gr_threshold_of(top, smp.r, merge.hop, row, merge.hop.graph ? *merge.maxnorm : 0.f);
}

// Element r (0 .. 15, different from lane to lane) of a lane's 16 accumulator values: a binary tree of selects on the
// bits of r.  (As assembly: written as conditional expressions the compiler turns the tree into a table in scratch
// memory that it indexes with r.  The s_nop after each compare: a select must not read a mask that one of the two
// instructions before it has written.)
__device__ __forceinline__ float gr_sym_pick16(const f32x16_t &a, int r) {
    float b0, b1, b2, b3, b4, b5, b6, b7, c0, c1, c2, c3, d0, d1, v;
    asm("v_and_b32 %8, 1, %25\n\tv_cmp_ne_u32 vcc, 0, %8\n\ts_nop 1\n\t"
        "v_cndmask_b32 %0, %9, %10, vcc\n\tv_cndmask_b32 %1, %11, %12, vcc\n\t"
        "v_cndmask_b32 %2, %13, %14, vcc\n\tv_cndmask_b32 %3, %15, %16, vcc\n\t"
        "v_cndmask_b32 %4, %17, %18, vcc\n\tv_cndmask_b32 %5, %19, %20, vcc\n\t"
        "v_cndmask_b32 %6, %21, %22, vcc\n\tv_cndmask_b32 %7, %23, %24, vcc"
        : "=&v"(b0), "=&v"(b1), "=&v"(b2), "=&v"(b3), "=&v"(b4), "=&v"(b5), "=&v"(b6), "=&v"(b7), "=&v"(v)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "v"(a[8]), "v"(a[9]),
          "v"(a[10]), "v"(a[11]), "v"(a[12]), "v"(a[13]), "v"(a[14]), "v"(a[15]), "v"(r)
        : "vcc");
    asm("v_and_b32 %4, 2, %13\n\tv_cmp_ne_u32 vcc, 0, %4\n\ts_nop 1\n\t"
        "v_cndmask_b32 %0, %5, %6, vcc\n\tv_cndmask_b32 %1, %7, %8, vcc\n\t"
        "v_cndmask_b32 %2, %9, %10, vcc\n\tv_cndmask_b32 %3, %11, %12, vcc"
        : "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3), "=&v"(v)
        : "v"(b0), "v"(b1), "v"(b2), "v"(b3), "v"(b4), "v"(b5), "v"(b6), "v"(b7), "v"(r)
        : "vcc");
    asm("v_and_b32 %2, 4, %7\n\tv_cmp_ne_u32 vcc, 0, %2\n\ts_nop 1\n\t"
        "v_cndmask_b32 %0, %3, %4, vcc\n\tv_cndmask_b32 %1, %5, %6, vcc"
        : "=&v"(d0), "=&v"(d1), "=&v"(v)
        : "v"(c0), "v"(c1), "v"(c2), "v"(c3), "v"(r)
        : "vcc");
    asm("v_and_b32 %0, 8, %3\n\tv_cmp_ne_u32 vcc, 0, %0\n\ts_nop 1\n\tv_cndmask_b32 %0, %1, %2, vcc"
        : "=&v"(v)
        : "v"(d0), "v"(d1), "v"(r)
        : "vcc");
    return v;
}

// The lane's hits among its 16 values as a bit mask, bit 15 - r for value r > t[r / 4][r % 4]: a compare and an
// add-with-carry per value.  (The four compares first: a vector instruction must not read a mask that one of the two
// instructions before it has written.)
__device__ __forceinline__ uint32_t gr_hit_mask4(uint32_t hm, float t0, float t1, float t2, float t3, float a0, float a1, float a2, float a3) {
    uint64_t k0, k1, k2, k3;
    asm("v_cmp_lt_f32 %1, %5, %9\n\tv_cmp_lt_f32 %2, %6, %10\n\tv_cmp_lt_f32 %3, %7, %11\n\t"
        "v_cmp_lt_f32 %4, %8, %12\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %1\n\tv_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %3\n\tv_addc_co_u32 %0, vcc, %0, %0, %4"
        : "+v"(hm), "=&s"(k0), "=&s"(k1), "=&s"(k2), "=&s"(k3)
        : "v"(t0), "v"(t1), "v"(t2), "v"(t3), "v"(a0), "v"(a1), "v"(a2), "v"(a3)
        : "vcc");
    return hm;
}
__device__ __forceinline__ uint32_t gr_hit_mask(float t, const f32x16_t &a) {
    uint32_t hm = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) hm = gr_hit_mask4(hm, t, t, t, t, a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
    return hm;
}

// Resident rows against one part of the searched rows.  Lane (row, half) appends to the row's segment of the part and
// counts in a register: an append is a store and an increment.  In the problems that come here one value in 30 to 1,000
// passes, so that of 64 lanes x 16 values nearly always some do: the hits of a lane become a bit mask and are taken one by
// one (testing value by value costs a branch around the append for each of them).
// TURNS: whether the halves of the workgroup take turns (ks_soe_pp_sweep).
template <int KT, bool RAGGED, class MERGE, bool TURNS>
__global__ void __launch_bounds__(512)
gr_recall_fix_kernel(GrPair pr, int D, int nb, int part_rows, GrSegs seg, MERGE merge, const float *__restrict__ thf_row,
                     uint64_t *__restrict__ cand, int32_t *__restrict__ cnt_res) {
    typedef typename std::conditional<TURNS, GrPp<KT, RAGGED>, GrSoe<KT, RAGGED>>::type CFG;
    __shared__ __attribute__((aligned(16))) uint16_t lds[CFG::LDS_ELEMS];
    const int id = ks_xcd_remap(blockIdx.x, gridDim.x); // the workgroups of an XCD stream the same parts
    const int part = id / nb;
    const int row0 = id % nb * CFG::RES;
    const int s0 = part * part_rows, s1 = (int64_t)s0 + part_rows < pr.Cs ? s0 + part_rows : (int)pr.Cs;
    const int Cr = (int)pr.Cr;
    const int cap = seg.cap(), last = 2 * seg.q - 1;
    const int64_t self0 = row0 + pr.self; // streamed rows [self0, self0 + RES) are this workgroup's own rows
    float thf;
    if constexpr (std::is_same<MERGE, GrMerge>::value) {
        const uint32_t bits = gr_merge_parts(merge, Cr, row0 + ks_soe_col());
        thf = row0 + ks_soe_col() < Cr ? gr_unorder(bits) : INFINITY;
        if (part == 0 && (threadIdx.x & 32) == 0 && row0 + ks_soe_col() < Cr) merge.tbits[row0 + ks_soe_col()] = bits;
    } else {
        thf = row0 + ks_soe_col() < Cr ? thf_row[row0 + ks_soe_col()] : INFINITY;
    }
    uint64_t *const wg_cand = cand + (int64_t)row0 * cap;
    // the lanes 0..31 fill their row's slots from the first one upwards, the lanes 32..63 from the last one downwards
    const int down = (threadIdx.x & 32) ? -1 : 0;
    const uint32_t my_base = (uint32_t)(ks_soe_col() * cap + 2 * part * seg.q + (down ? last + 1 : 0));
    int my_cnt = 0;
    // A lane finds half of the rows at most; one that may run out of slots here stores nothing any more, and its count, which
    // no segment holds, marks the row as overflowed.
    auto threshold_with_room = [&](int rows) __attribute__((always_inline)) {
        if (my_cnt > last + 1 - rows / 2) my_cnt = 1 << 20;
        return my_cnt >= 1 << 20 ? INFINITY : thf;
    };
    auto special = [&](int c0, int rows_here) __attribute__((always_inline)) { // a chunk with rows beyond the part's last, or own rows
        return rows_here < CFG::CH || ((int64_t)c0 < self0 + CFG::RES && (int64_t)c0 + CFG::CH > self0);
    };
    auto no_hits = [&](int first, int end, uint32_t hm) __attribute__((always_inline)) { // without rows from `end` on and the row itself
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int j = first + 8 * (r >> 2) + (r & 3);
            if (j >= end || (int64_t)j == (int64_t)row0 + ks_soe_col() + pr.self) hm &= ~(0x8000u >> r);
        }
        return hm;
    };
    auto key = [&](float v, int j) __attribute__((always_inline)) { return ((uint64_t)gr_orderable(v) << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)j); };
    if constexpr (TURNS) {
        auto epi = [&](auto block, int c0, int rows_here, const f32x16_t &acc) __attribute__((always_inline)) {
            uint32_t hm = gr_hit_mask(threshold_with_room(32), acc);
            int first = c0 + 32 * decltype(block)::value + 4 * ((threadIdx.x >> 5) & 1);
            asm volatile("" : "+v"(first));
            if (special(c0, rows_here)) hm = no_hits(first, c0 + rows_here, hm);
            while (__ballot(hm != 0u) != 0ull) { // as often as the lane with the most hits has some
                const int r = 15 - (__ffs(hm) - 1);
                const float v = gr_sym_pick16(acc, r);
                const int j = first + r + (r & 12);
                if (hm != 0u) wg_cand[my_base + (uint32_t)(my_cnt ^ down)] = key(v, j);
                my_cnt += hm != 0u ? 1 : 0;
                hm &= hm - 1u;
            }
        };
        ks_soe_pp_sweep<CFG>(pr.R, D, row0, Cr, pr.S, D, s0, s1, (int)pr.Cs, lds, epi);
    } else {
        // (Here a whole chunk's values are at hand, and what is the same for all of them is worked out once; with the loop above,
        // block by block: 150,000 x 64, K = 32: 5.18 ms -> 5.57.)
        auto chunk = [&](int c0, int rows_here, f32x16_t (&acc)[CFG::FM]) __attribute__((always_inline)) {
            const float t = threshold_with_room(CFG::CH);
            const bool check = special(c0, rows_here);
            auto one = [&](auto block) __attribute__((always_inline)) {
                constexpr int f = decltype(block)::value;
                uint32_t hm = gr_hit_mask(t, acc[f]);
                const int first = c0 + 32 * f + 4 * ((threadIdx.x >> 5) & 1);
                if (check) hm = no_hits(first, c0 + rows_here, hm);
                while (__ballot(hm != 0u) != 0ull) {
                    if (hm != 0u) {
                        const int r = 15 - __builtin_ctz(hm);
                        hm &= hm - 1u;
                        const float v = gr_sym_pick16(acc[f], r);
                        wg_cand[my_base + (uint32_t)(my_cnt ^ down)] = key(v, first + r + (r & 12));
                        ++my_cnt;
                    }
                }
            };
            ks_each<CFG::FM>(one);
        };
        ks_soe_sweep<CFG>(pr.R, D, row0, Cr, pr.S, D, nullptr, s0, s1, (int)pr.Cs, lds, chunk);
    }
    const int i = row0 + ks_soe_col();
    if (i < Cr) cnt_res[(int64_t)i * 2 * seg.parts + 2 * part + ((threadIdx.x & 63) >> 5)] = my_cnt;
}

// ------------------------------------------------------------------------------------------------
// recall pass that computes every similarity ONCE (W searched in W, D = 128, 256 or 512, K <= 64).
//
// The similarity matrix is symmetric, so the tile of a workgroup's 256 resident rows against a streamed row j holds,
// for every resident row i, a candidate for BOTH lists: j for row i (the "resident side", a lane's own row, as in the
// kernel above) and i for row j (the "stream side").  Each unordered pair of 256-row blocks is given to exactly one
// share of the work, which halves the MFMA work of the pass.  What it takes beyond the fixed thresholds:
//
//  * who takes which pair.  Rows are cut into blocks of 256 (a share's resident rows), super-blocks of 768 rows
//    (three blocks, and whole chunks of every size, so that every streamed range starts on a chunk boundary) and groups of up
//    to 10 super-blocks.  On each level the members form a ring and a member takes the following half of the ring
//    (gr_sym_succ): a share streams its own super-block (its own block for the resident side only, the blocks it
//    takes there for both sides), then the super-blocks it takes inside its group, then all rows of the groups its
//    group takes.  A share's chunks are cut into `parts` runs, one workgroup each (one part per share in problems that
//    fill the chip without it).  The shares of a group run on one XCD (or two neighbouring ones) and stream the same long
//    ranges, so a streamed row is fetched from memory about once per group -- less often where two groups that stream
//    different ranges share an XCD (390,625 rows of 512: 31.6 GB in all, 26.3 when whole groups were dealt to XCDs).
//  * the stream side's candidates.  A hit for streamed row j is a record (j, i, similarity): a wavefront collects them
//    in LDS and appends them, with one atomic per batch, to the log of j's run of `log_rows` rows (a super-block, or half
//    of one in a smaller problem); gr_sym_scatter_kernel (one workgroup per log, row counters in LDS) then moves them into the rows' stream segments.
//  * A row whose segments or log overflowed gets a threshold no similarity exceeds: its certificate fails and the
//    exhaustive pass computes it.
// ------------------------------------------------------------------------------------------------
#define GR_SYM_SB 768            /* rows of a super-block */
// Log records per row: what a row's stream segment takes.  Half of a row's hits are stream-side ones where its neighbours lie
// anywhere; but where they crowd in a run of ids (classes in order of frequency, with norms to match), the rows of the half
// ring behind that run find ALL of theirs on the stream side, and all the same ones: the mean of a log is then a single
// order statistic, beyond 384 for one build in four at K = 32 and for half of them at K = 64.  One lost record sends all
// rows of the log to the exhaustive search.
#define GR_SYM_LOG_PER_ROW GR_SYM_SCAP
#define GR_SYM_STAGE 192         /* records a wavefront collects in LDS between two appends to a log */
#define GR_SYM_MAX_GROUP 10      /* super-blocks per group at most: 30 shares, about the compute units of an XCD */

// members of a ring of n that member x takes: the next gr_sym_succ(n, x) ones.  Every unordered pair is taken once:
// for even n the opposite member is taken by the lower of the two.
__host__ __device__ __forceinline__ int gr_sym_succ(int n, int x) {
    return (n & 1) ? (n - 1) / 2 : (x < n / 2 ? n / 2 : n / 2 - 1);
}
__host__ __device__ __forceinline__ int gr_sym_group_sbs(int64_t C) { // super-blocks per group
    const int nsb = (int)((C + GR_SYM_SB - 1) / GR_SYM_SB);
    const int gs = nsb / 16;
    return gs < 1 ? 1 : (gs > GR_SYM_MAX_GROUP ? GR_SYM_MAX_GROUP : gs);
}

// The plan of the sweep, made by a small kernel beforehand (the sweep kernel has no registers to spare for the
// arithmetic).  Per workgroup GR_SYM_PLAN words: [0] the resident block or -1, [1] the block's place in the ring of its
// super-block's blocks (place | members << 4 | members it takes << 8), [2] the number of chunks it streams; and a table
// of those chunks (first row, rows): its own super-block, then the super-blocks it takes in its group (two ranges: the
// ring wraps), then the groups its group takes (likewise).
#define GR_SYM_PLAN 4
struct GrSymRanges {
    int block;          // resident block, or -1: the workgroup has none
    int ring;           // place | members << 4 | members taken << 8 in the ring of its super-block's blocks
    int first[5], end[5]; // streamed rows [first, end) of the five ranges; empty: end <= first
};
__host__ __device__ inline GrSymRanges gr_sym_ranges(int block, int C, int GS) {
    GrSymRanges out;
    const int NB = (C + 255) / 256, NSB = (C + GR_SYM_SB - 1) / GR_SYM_SB, NG = (NSB + GS - 1) / GS;
    const int g = block / (GS * (GR_SYM_SB / 256));
    out.block = -1;
    out.ring = 0;
    for (int part = 0; part < 5; ++part) out.first[part] = out.end[part] = 0;
    if (block >= NB) return out;
    const int sb = block * 256 / GR_SYM_SB, own0 = sb * GR_SYM_SB, own1 = own0 + GR_SYM_SB < C ? own0 + GR_SYM_SB : C;
    const int kb = (block * 256 - own0) / 256, n_b = (own1 - own0 + 255) / 256;
    const int gsb0 = g * GS, n_sb = (gsb0 + GS < NSB ? gsb0 + GS : NSB) - gsb0, s_loc = sb - gsb0;
    const int succ_s = gr_sym_succ(n_sb, s_loc), succ_g = gr_sym_succ(NG, g);
    out.block = block;
    out.ring = kb | (n_b << 4) | (gr_sym_succ(n_b, kb) << 8);
    for (int part = 0; part < 5; ++part) {
        int b = 0, e = 0; // in super-blocks
        if (part == 0) { b = sb; e = sb + 1; }
        else if (part == 1) { b = sb + 1; e = gsb0 + (s_loc + succ_s < n_sb - 1 ? s_loc + succ_s : n_sb - 1) + 1; }
        else if (part == 2) { b = gsb0; e = gsb0 + (s_loc + succ_s - n_sb) + 1; }
        else if (part == 3) { b = (g + 1) * GS; e = ((g + succ_g < NG - 1 ? g + succ_g : NG - 1) + 1) * GS; }
        else { b = 0; e = (g + succ_g - NG + 1) * GS; }
        if (e > NSB) e = NSB;
        if (e <= b) continue;
        const long long e_row = (long long)e * GR_SYM_SB;
        out.first[part] = b * GR_SYM_SB;
        out.end[part] = e_row < C ? (int)e_row : C;
    }
    return out;
}
__global__ void __launch_bounds__(GR_NT)
gr_sym_plan_kernel(int C, int GS, int ch, int32_t *__restrict__ plan, int2 *__restrict__ chunks, int chunks_stride) {
    const int wg = blockIdx.x;
    int32_t *out = plan + (int64_t)wg * GR_SYM_PLAN;
    int2 *tab = chunks + (int64_t)wg * chunks_stride;
    const GrSymRanges r = gr_sym_ranges(wg, C, GS);
    int n_chunks = 0;
    for (int part = 0; part < 5; ++part) {
        if (r.end[part] <= r.first[part]) continue;
        const int n = (r.end[part] - r.first[part] + ch - 1) / ch;
        for (int c = threadIdx.x; c < n; c += GR_NT) {
            const int first = r.first[part] + c * ch;
            if (n_chunks + c < chunks_stride) tab[n_chunks + c] = make_int2(first, r.end[part] - first < ch ? r.end[part] - first : ch);
        }
        n_chunks += n;
    }
    if (threadIdx.x == 0) {
        out[0] = r.block;
        out[1] = r.ring;
        out[2] = n_chunks < chunks_stride ? n_chunks : chunks_stride; // (the stride is sized for the longest plan)
    }
}

// a stream-side hit: similarity v of a streamed row (given by its place in its super-block) with resident row `other`
__device__ __forceinline__ uint2 gr_sym_record(int j_in_sb, int other, float v) {
    return make_uint2(gr_orderable(v), ((uint32_t)other << 10) | (uint32_t)j_in_sb);
}

// SPLIT: shares are cut into parts and the logs are finer than a super-block (the addresses are then arithmetic on two
// more registers; compiled apart, the sweep over 390,625 rows of 512 takes 84 ms instead of 88).
template <int KT, bool SPLIT>
__global__ void __launch_bounds__(512)
gr_recall_sym_kernel(const uint16_t *__restrict__ W, int C, int D, const int32_t *__restrict__ plan,
                     const int2 *__restrict__ chunks, int chunks_stride, int split_parts, int split_log_rows,
                     const float *__restrict__ thf_row, uint64_t *__restrict__ cand, int32_t *__restrict__ cnt_res,
                     uint2 *__restrict__ log, int32_t *logcnt) {
    typedef GrPp<KT, false> CFG;
    constexpr int Q = GR_SYM_Q, SB = GR_SYM_SB;
    const int parts = SPLIT ? split_parts : 1, log_rows = SPLIT ? split_log_rows : SB;
    static_assert(SB % CFG::CH == 0 && SB % CFG::RES == 0 && CFG::RES == 256, "super-blocks are whole chunks and whole blocks");
    static_assert(SB / 2 % CFG::CH == 0, "a log of half a super-block is whole chunks");
    // one LDS array (see ks_gemm_soe.h): the stream stages, the streamed rows' thresholds of the chunks in flight, the
    // records that the wavefronts collect
    constexpr int THR_ELEMS = 2 * 8 * CFG::CH, STAGE_ELEMS = 4 * GR_SYM_STAGE;
    __shared__ __attribute__((aligned(16))) uint16_t lds[CFG::LDS_ELEMS + THR_ELEMS + CFG::NW * STAGE_ELEMS];
    float(*const s_thr)[CFG::CH] = (float(*)[CFG::CH])(lds + CFG::LDS_ELEMS);
    const int lane = threadIdx.x & 63;
    // Share and part.  Every XCD gets the same number of workgroups, for consecutive blocks: the 32 that it runs at a time
    // belong to one group and the next.  (Whole groups dealt to XCDs: at 390,625 rows three XCDs had seven groups of 30
    // and five had six, seven rounds of workgroups instead of six, 87 ms instead of 75.)
    const int id = ks_xcd_remap(blockIdx.x, gridDim.x), shares = (int)gridDim.x / parts, share = id % shares, part = id / shares;
    const int32_t *my_plan = plan + (int64_t)share * GR_SYM_PLAN;
    const int block = my_plan[0];
    if (block < 0) return;
    const int chunk0 = (int)((int64_t)my_plan[2] * part / parts), chunk1 = (int)((int64_t)my_plan[2] * (part + 1) / parts);
    const int row0 = block * CFG::RES;
    const int sb_own = row0 / SB;
    const int ring = my_plan[1];
    const float thf = row0 + ks_soe_col() < C ? thf_row[row0 + ks_soe_col()] : INFINITY;
    const int cap = 2 * Q * parts + GR_SYM_SCAP;
    uint64_t *const wg_cand = cand + (int64_t)row0 * cap;
    int my_cnt = 0;
    // stream side: records collected by this wavefront, and the log they belong to (log_rows is a multiple of the chunk
    // and divides the super-block)
    int staged = 0, cur_log = -1;
    auto my_stage = [&]() __attribute__((always_inline)) {
        return (uint2 *)(lds + CFG::LDS_ELEMS + THR_ELEMS + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * STAGE_ELEMS);
    };
    auto flush = [&]() {
        if (staged > 0) {
            int base = 0;
            if (lane == 0) base = atomicAdd(&logcnt[cur_log], staged);
            base = __builtin_amdgcn_readfirstlane(base);
            const int logcap = log_rows * GR_SYM_LOG_PER_ROW;
            uint2 *dst = log + (int64_t)cur_log * logcap;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the records written by the other lanes are in LDS
            for (int q = lane; q < staged; q += 64)
                if (base + q < logcap) dst[base + q] = my_stage()[q];
            asm volatile("" ::: "memory");
            staged = 0;
        }
    };
    auto append_res = [&](int j, float v) __attribute__((always_inline)) {
        // (the mask keeps the store inside the lane's half; a count beyond Q marks the row as overflowed)
        const uint32_t my_base = (uint32_t)(ks_soe_col() * cap + (2 * part + (lane >> 5)) * Q);
        wg_cand[my_base + ((uint32_t)my_cnt & (uint32_t)(Q - 1))] = ((uint64_t)gr_orderable(v) << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)j);
        ++my_cnt;
    };
    // The thresholds of a chunk's rows travel to LDS beside its rows: requested by wavefront 0 when the chunk's loads begin.
    // The loads run up to STAGES - 1 pipeline stages ahead of the MFMAs and the epilogue a chunk behind them: AHEAD chunks at most (six at
    // D = 128, where a chunk is a single stage) from the request to the epilogue that reads it, and eight slots.
    static_assert(CFG::AHEAD <= 8, "slots for the chunks in flight");
    auto side = [&](int first, int c) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < CFG::CH; u += 64)
            if (u + 64 <= CFG::CH || lane < CFG::CH - u)
                __builtin_amdgcn_global_load_lds(KS_GPTR(thf_row + first + u + lane), KS_LPTR(&s_thr[c & 7][u]), 4, 0, 0);
    };
    int epi_chunk = 0; // chunks seen by the epilogue: the slot of their thresholds
    auto epi = [&](auto block32, int c0, int rows_here, const f32x16_t &acc) __attribute__((always_inline)) {
        constexpr int fm = decltype(block32)::value;
        const float *thr_chunk = s_thr[epi_chunk & 7];
        if (fm == CFG::FM - 1) ++epi_chunk;
        const int sb = c0 / SB; // uniform; a chunk lies in one super-block and in one log
        if (fm == 0 && (c0 < cur_log * log_rows || c0 >= (cur_log + 1) * log_rows)) { flush(); cur_log = c0 / log_rows; }
        // Which sides are wanted is the same for 32 streamed rows at a time (block boundaries are multiples of 32 rows):
        // both, except in the workgroup's own super-block, where its own block is searched for the resident side only and
        // the other blocks as the ring says.
        const bool own_sb = sb == sb_own, ragged = rows_here < CFG::CH; // (ragged: the last chunk of W)
        const bool real_row = row0 + ks_soe_col() < C;
        {
            bool res_side = true, str_side = true, diag = false;
            if (own_sb) {
                const int kb = ring & 15, n_b = (ring >> 4) & 15, succ_b = ring >> 8;
                int dd = (c0 + fm * 32 - sb_own * SB) / CFG::RES - kb; // ring distance from this block to the streamed rows' block
                if (dd < 0) dd += n_b;
                diag = dd == 0;
                str_side = dd >= 1 && dd <= succ_b;
                res_side = diag || str_side;
            }
            if (res_side) {
                const bool check = diag || ragged;
                if (SPLIT) {
                    uint32_t hr = gr_hit_mask(thf, acc);
                    int first = c0 + fm * 32 + 4 * (lane >> 5);
                    asm volatile("" : "+v"(first));
                    if (check) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int j = first + 8 * (r >> 2) + (r & 3);
                            if (j >= c0 + rows_here || j == row0 + ks_soe_col()) hr &= ~(0x8000u >> r);
                        }
                    }
                    while (__ballot(hr != 0u) != 0ull) {
                        const int r = 15 - (__ffs(hr) - 1);
                        const float v = gr_sym_pick16(acc, r);
                        if (hr != 0u) append_res(first + r + (r & 12), v);
                        hr &= hr - 1u;
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) { // four values at a time: most groups have none that passes
                        const float a0 = acc[4 * q], a1 = acc[4 * q + 1], a2 = acc[4 * q + 2], a3 = acc[4 * q + 3];
                        if (fmaxf(fmaxf(a0, a1), fmaxf(a2, a3)) > thf) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float v = acc[4 * q + e];
                                if (v > thf) {
                                    const int lr = ks_soe_row(fm, 4 * q + e, lane);
                                    if (!check || (lr < rows_here && c0 + lr != row0 + ks_soe_col())) append_res(c0 + lr, v);
                                }
                            }
                        }
                    }
                }
            }
            if (str_side) {
                // Stream side.  An accumulator register holds ONE streamed row in the lanes 0..31 and the row four further
                // on in the lanes 32..63.  (Testing against the smaller of the two thresholds, held in a scalar register,
                // and sorting out the surplus later was tried: the number of records then depends on how well
                // neighbouring rows match; a tight cluster row beside a lone one got four times its share, the logs
                // overflowed and every row went to the exhaustive pass.  With the exact test a row's hits on both
                // sides together are the sample's order statistic and nothing else.)
                // Every instruction here runs once per chunk and fragment, so there are few: a lane's hits become a bit
                // mask (bit 15 - r for element r); while any lane has a hit left, every lane that has picks one with a
                // binary tree of selects and the slots come from one ballot.
                // (a lane reads the four thresholds of its own rows from LDS: rows 8 q + e in the lanes 0..31, 8 q + 4 + e
                // in the lanes 32..63)
                uint32_t hm = 0u;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4_t t4 = *(const f32x4_t *)(thr_chunk + fm * 32 + 8 * q + 4 * (lane >> 5));
                    hm = gr_hit_mask4(hm, t4[0], t4[1], t4[2], t4[3], acc[4 * q], acc[4 * q + 1], acc[4 * q + 2],
                                      acc[4 * q + 3]);
                }
                if (!real_row) hm = 0u; // (streamed rows beyond W have a threshold that nothing exceeds)
                uint64_t any = __ballot(hm != 0u);
                while (any != 0ull) {
                    const int n = __popcll(any);
                    if (staged + n > GR_SYM_STAGE) flush();
                    const int r = 15 - (__ffs(hm) - 1);
                    const float v = gr_sym_pick16(acc, r);
                    const int lr = fm * 32 + 4 * (lane >> 5) + r + (r & 12);
                    if (hm != 0u)
                        my_stage()[staged + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(any >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)any, 0u))] =
                            gr_sym_record(c0 - cur_log * log_rows + lr, row0 + ks_soe_col(), v);
                    hm &= hm - 1u;
                    staged = __builtin_amdgcn_readfirstlane(staged + n);
                    any = __ballot(hm != 0u);
                }
            }
        }
    };
    ks_soe_pp_sweep<CFG>(W, D, row0, C, W, D, 0, 0, C, lds, epi, chunks + (int64_t)share * chunks_stride + chunk0, chunk1 - chunk0, side);
    flush();
    if (row0 + ks_soe_col() < C)
        cnt_res[(int64_t)(row0 + ks_soe_col()) * 2 * parts + 2 * part + (lane >> 5)] = my_cnt;
}

// the stream-side records of a log go to the rows they belong to; one workgroup per log
__global__ void __launch_bounds__(1024)
gr_sym_scatter_kernel(const uint2 *__restrict__ log, const int32_t *__restrict__ logcnt, int C, int log_rows, GrSegs seg,
                      uint64_t *__restrict__ cand, int32_t *__restrict__ cnt_str) {
    __shared__ int s_cnt[GR_SYM_SB];
    const int row0 = blockIdx.x * log_rows, logcap = log_rows * GR_SYM_LOG_PER_ROW, cap = seg.cap();
    for (int r = threadIdx.x; r < log_rows; r += 1024) s_cnt[r] = 0;
    __syncthreads();
    const int n_raw = logcnt[blockIdx.x], n = n_raw < logcap ? n_raw : logcap;
    const uint2 *src = log + (int64_t)blockIdx.x * logcap;
    for (int q0 = 0; q0 < n; q0 += 4 * 1024) { // four records per thread in flight
        uint2 rec[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = q0 + u * 1024 + (int)threadIdx.x;
            rec[u] = q < n ? src[q] : make_uint2(0u, 0xFFFFFFFFu); // (place 1023 of a log: dropped below)
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jl = (int)(rec[u].y & 1023u); // (checked all the same: it becomes an address)
            const uint32_t other = rec[u].y >> 10;
            if (jl >= log_rows || row0 + jl >= C || other >= (uint32_t)C) continue;
            const int slot = atomicAdd(&s_cnt[jl], 1);
            if (slot < seg.stream)
                cand[(int64_t)(row0 + jl) * cap + 2 * seg.parts * seg.q + slot] = ((uint64_t)rec[u].x << 32) | (uint32_t)(0xFFFFFFFFu - other);
        }
    }
    __syncthreads();
    for (int r = threadIdx.x; r < log_rows; r += 1024)
        if (row0 + r < C) cnt_str[row0 + r] = n_raw > logcap ? 0x7FFFFFFF : s_cnt[r]; // a lost record: all rows overflow
}

// ------------------------------------------------------------------------------------------------
// canonical similarity: sum over d ascending of (double)a_d * (double)b_d, one fused multiply-add per
// term (the product of two fp32 or bf16 values is exact in fp64, so this equals multiply-then-add)
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ double gr_canon(const uint16_t *__restrict__ a, const uint16_t *__restrict__ b, int D) {
    double acc = 0.0;
    int d = 0;
    // whole 128-byte lines of b at a time: callers give every lane a row of its own, so a line that is only
    // partly consumed is evicted before the lane comes back to it and is fetched again
    for (; d + 64 <= D; d += 64) {
        uint4 vb[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) vb[q] = *(const uint4 *)(b + d + q * 8);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint4 va = *(const uint4 *)(a + d + q * 8);
            const uint32_t wa[4] = {va.x, va.y, va.z, va.w}, wb[4] = {vb[q].x, vb[q].y, vb[q].z, vb[q].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc = __builtin_fma((double)__uint_as_float(wa[e] << 16), (double)__uint_as_float(wb[e] << 16), acc);
                acc = __builtin_fma((double)__uint_as_float(wa[e] & 0xFFFF0000u),
                                    (double)__uint_as_float(wb[e] & 0xFFFF0000u), acc);
            }
        }
    }
    for (; d < D; d += 8) {
        uint4 va = *(const uint4 *)(a + d), vb = *(const uint4 *)(b + d);
        const uint32_t wa[4] = {va.x, va.y, va.z, va.w}, wb[4] = {vb.x, vb.y, vb.z, vb.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc = __builtin_fma((double)__uint_as_float(wa[e] << 16), (double)__uint_as_float(wb[e] << 16), acc);
            acc = __builtin_fma((double)__uint_as_float(wa[e] & 0xFFFF0000u), (double)__uint_as_float(wb[e] & 0xFFFF0000u),
                                acc);
        }
    }
    return acc;
}
__device__ __forceinline__ double gr_canon(const float *__restrict__ a, const float *__restrict__ b, int D) {
    double acc = 0.0;
    for (int d = 0; d < D; d += 32) { // whole 128-byte lines of b at a time, as above (D % 32 == 0)
        float4 vb[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) vb[q] = *(const float4 *)(b + d + q * 4);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float4 va = *(const float4 *)(a + d + q * 4);
            acc = __builtin_fma((double)va.x, (double)vb[q].x, acc);
            acc = __builtin_fma((double)va.y, (double)vb[q].y, acc);
            acc = __builtin_fma((double)va.z, (double)vb[q].z, acc);
            acc = __builtin_fma((double)va.w, (double)vb[q].w, acc);
        }
    }
    return acc;
}

__device__ __forceinline__ bool gr_ranks_before(double s, int32_t j, double t, int32_t k) {
    return s > t || (s == t && j < k);
}
// the value that lane `src` (uniform) holds, in scalar registers
__device__ __forceinline__ double gr_readlane(double v, int src) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, src), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), src);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
#define GR_NO_ID 0x7FFFFFFF
// rank[t] += the number of the first n (<= 64) lanes' entries (s2, id2) that rank before the lane's entry t
template <int S>
__device__ __forceinline__ void gr_count_before(double s2, int32_t id2, int n, const double (&s)[S], const int32_t (&id)[S], int (&rank)[S]) {
    for (int src = 0; src < n; ++src) {
        const double os = gr_readlane(s2, src);
        const int32_t oid = __builtin_amdgcn_readlane(id2, src);
#pragma unroll
        for (int t = 0; t < S; ++t) rank[t] += gr_ranks_before(os, oid, s[t], id[t]) ? 1 : 0;
    }
}

// ------------------------------------------------------------------------------------------------
// exact ranking of the candidates; one wavefront per row, at most 64 * KP candidates ranked
//
// Build (HOP false): first K of the row's candidates.  Hop (HOP true): best K of candidates and list so far (ids of the
// whole problem = visit_offset + row); a candidate that is in the list already is dropped.
//
// Ranked are the candidates whose 16-bit similarity lies no more than 2.5 error bounds below the K-th largest: K of them
// are at least (K-th largest - bound) exactly, and what is left out is at most (that - 1.5 bounds).  That is K and a few
// for bf16 rows (K and 16 or more were ranked before: 19.7 GB of gathered rows at 390,625 x 512, K = 32).  Where more than
// 64 * KP lie that close, the best 64 * KP are ranked, and the certificate decides.
// One kernel does what were three passes over the candidates (cut, re-rank, and before them a gather of the
// segments): the keys are read once, and the row's own data and the other lanes' entries come through scalar registers
// (the ranking by shuffles cost three LDS permutes and 24 instructions per entry, now three lane reads and 6).
// The kernel is bound by the instructions it issues.  Where a key lies in the segments comes from a running sum over LDS (before, a
// loop over the segments for every register of keys), and for K <= 32 the K-th key is first bounded by the lanes' largest values, one
// compare a round, and then searched among the at most 64 keys above the bound (before, 4 or 8 compares a round).  Builds, us:
// 2,000 x 64, K = 16: 41.2 -> 33.1; 10,000 x 128, K = 8, fp32: 119.0 -> 113.8; 8,000 x 320, K = 24: 119 -> 114; two hops of 15,000 x 15,000
// x 256, K = 32: 500 -> 491.
// (Not for K > 32, where rows are few wavefronts and the chain of LDS accesses counts: 2,600 x 512, K = 64, fp32: 146 -> 153.  Five
// wavefronts to a SIMD for K <= 32: 5,000 x 320, K = 32, fp32: 128 with four, 122.5.)
// LANES: with that bound and the running sum.  Not for fp32 rows with K > 29 and D > 128: the K-th of 64 largest values is nearly their
// median, similarities of longer rows lie closer together while the error bound is that of rounding the rows, and more than 64
// keys are above the bound so often that the first search is wasted.  K = 32, plain, by lanes: 2,600 x 320 83.5 us, 85.5; 4,500 x
// 320 120, 125; 4,900 x 256 106, 109; 20,000 x 256 423, 431; but 5,800 x 512 187, 182; 4,200 x 64 70.2, 63.6; K = 29: 900 x 320 58.2, 52.0;
// a hop of 120 x 2,909 x 192 67.2, 61.9.
// SHORT: lists of at most 256 candidates have a copy of the search of their own, taken for K <= 24 (beyond, too few rows have
// so few).  For K <= 32 the kernel of K > 24 does without the copy, which alone costs it 1 %; so does that of K <= 24 where few rows
// gain by it, those of fp32 builds and of hops (one row in 32 sampled), and the rows are one round of the chip (2,000 x 256, K = 16,
// fp32: 64.3 -> 63.3 us; 5,000 x 512, K = 16, fp32, with it: 134 -> 130).  For K > 32 and bf16 rows the
// compiler needs 83 registers with it and 123 without: five wavefronts to a SIMD instead of four, but the longer chain of one.
// So it has the copy where the rows need more than one round of the chip at four (GR_RANK_AT_ONCE).  Builds, us, without -> with:
// 2,000 x 512, K = 64: 87.3 -> 88.6; 4,000 x 320, K = 33: 92.2 -> 93.0; 5,000 x 512, K = 64: 162.9 -> 149.4; 20,000 x 64, K = 64: 319 -> 301.
// ------------------------------------------------------------------------------------------------
#define GR_RANK_AT_ONCE 4096 /* 256 compute units x 4 workgroups x 4 rows */
template <typename IN, int KP, bool HOP, bool SHORT, bool LANES>
__global__ void __launch_bounds__(GR_NT, KP == 1 ? 5 : 4)
gr_rank_kernel(const IN *__restrict__ Wl, int64_t C, const IN *__restrict__ Wv, int64_t Cv, int D, int K, GrSegs seg,
               const uint64_t *__restrict__ cand, const int32_t *__restrict__ cnt_res, const int32_t *__restrict__ cnt_str,
               const uint32_t *__restrict__ tbits, const float *__restrict__ norms, const float *__restrict__ maxnorm, float gamma,
               int64_t visit_offset, int32_t *__restrict__ graph, void *__restrict__ sims_, int32_t *list_count,
               int32_t *__restrict__ list_rows) {
    __shared__ uint64_t s_key[GR_NT / 64][KP * 64];
    __shared__ int s_grow[GR_NT / 64][512];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * (GR_NT / 64) + wave;
    if (i >= C) return;
    // the row's segments: lane s looks at segment s
    const int nseg = 2 * seg.parts + (seg.stream > 0 ? 1 : 0);
    int c, begin;
    bool overflow = gr_segments(seg, cnt_res, cnt_str, i, c, begin);
    const int incl = ks_wave_iscan(c), excl = incl - c, shift = begin - excl;
    int n = __builtin_amdgcn_readlane(incl, 63);
    if (n > GR_MAX_CAND) { n = GR_MAX_CAND; overflow = true; }
    const uint32_t tb = tbits[i];
    const uint64_t *__restrict__ row = cand + i * seg.cap();
    const double eps = (double)gamma * (double)norms[i] * (double)*maxnorm; // error bound of the 16-bit similarities
    uint32_t thr = tb; // nothing above this value (as a key) was dropped
    int kept = n;
    // The keys to rank to LDS.  E: registers for the keys.  The m-th largest value by a bitwise search ("how many keys are
    // >= this prefix": a compare, a ballot and a population count per register and round) below the bits that threshold
    // and largest key share; it ends as soon as exactly m keys are left (a bound below the m-th and above the next).
    auto select = [&](auto e_) __attribute__((always_inline)) {
        constexpr int E = decltype(e_)::value;
        uint64_t val[E];
        // (an index counts through the segments laid end to end: what has to be added to it to find its place grows at the first index
        // of every segment)
        if (LANES && E <= 8 && nseg > 4) {
            int *const grow = s_grow[wave];
#pragma unroll
            for (int r = 0; r < E; ++r) grow[r * 64 + lane] = 0;
            asm volatile("" ::: "memory");
            const int before = __shfl_up(shift, 1, 64);
            if (lane > 0 && lane < nseg && excl < n) atomicAdd(&grow[excl], shift - before);
            asm volatile("" ::: "memory"); // (a wavefront's LDS instructions are carried out in order)
            int carry = 0; // (the first segment begins at 0)
#pragma unroll
            for (int r = 0; r < E; ++r) {
                val[r] = 0ull; // below every real key
                if (r * 64 < n) {
                    const int adj = ks_wave_iscan(grow[r * 64 + lane]) + carry;
                    carry = __builtin_amdgcn_readlane(adj, 63);
                    if (r * 64 + lane < n) val[r] = row[r * 64 + lane + adj];
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < E; ++r) {
                val[r] = 0ull;
                if (r * 64 < n) {
                    const int idx = r * 64 + lane;
                    int adj = 0;
                    for (int sg = 1; sg < nseg; ++sg) {
                        const int st = __builtin_amdgcn_readlane(excl, sg);
                        const int sh = __builtin_amdgcn_readlane(shift, sg);
                        if (idx >= st) adj = sh;
                    }
                    if (idx < n) val[r] = row[idx + adj];
                }
            }
        }
        // the keys for which keep(value) holds go to the front of LDS; returns how many (64 KP at most are stored)
        auto compact = [&](auto keep) __attribute__((always_inline)) {
            int base = 0;
#pragma unroll
            for (int r = 0; r < E; ++r) {
                if (r * 64 < n) {
                    const bool k = r * 64 + lane < n && keep(val[r]);
                    const uint64_t m = __ballot(k);
                    const int q = base + __popcll(m & ((1ull << lane) - 1ull));
                    if (k && q < KP * 64) s_key[wave][q] = val[r];
                    base += __popcll(m);
                }
            }
            return base;
        };
        uint64_t t = 1ull; // keeps every real key
        if (n > K) {
            auto count_hi = [&](uint32_t v) __attribute__((always_inline)) {
                int k = 0;
#pragma unroll
                for (int r = 0; r < E; ++r)
                    if (E <= 8 || r * 64 < n) k += __popcll(__ballot((uint32_t)(val[r] >> 32) >= v));
                return k;
            };
            uint32_t mine = 0u; // the largest value of the lane
#pragma unroll
            for (int r = 0; r < E; ++r) mine = (uint32_t)(val[r] >> 32) > mine ? (uint32_t)(val[r] >> 32) : mine;
            uint32_t mx = mine;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const uint32_t other = (uint32_t)__shfl_xor((int)mx, o, 64);
                mx = other > mx ? other : mx;
            }
            mx = (uint32_t)__builtin_amdgcn_readfirstlane((int)mx);
            const int top_bit = mx > tb ? 31 - __builtin_clz(mx ^ tb) : -1; // (always above: only such keys are appended)
            const uint32_t prefix = top_bit >= 31 ? 0u : (top_bit < 0 ? mx : mx >> (top_bit + 1) << (top_bit + 1));
            auto search_by = [&](int m, bool &exact, auto count) __attribute__((always_inline)) {
                uint32_t v = prefix;
                exact = false;
                for (int bit = top_bit; bit >= 0 && !exact; --bit) {
                    const int k = count(v | (1u << bit));
                    if (k >= m) v |= 1u << bit;
                    exact = k == m;
                }
                return v;
            };
            auto search = [&](int m, bool &exact) __attribute__((always_inline)) { return search_by(m, exact, count_hi); };
            auto below = [&](uint32_t v) __attribute__((always_inline)) { // 2.5 error bounds lower
                const double low = (double)gr_unorder(v) - 2.5 * eps;
                float f = (float)low;
                if ((double)f > low) f = nextafterf(f, -INFINITY); // rounded down
                return f == f ? gr_orderable(f) : 0u;
            };
            bool exact;
            if (LANES) {
                // The K-th largest of the lanes' largest values is a bound that K keys reach, found with one compare a round instead of E;
                // what lies above it (less 2.5 error bounds) is a key per lane, and the search goes on among those.
                const uint32_t bound = below(search_by(K, exact, [&](uint32_t v) __attribute__((always_inline)) { return __popcll(__ballot(mine >= v)); }));
                const int few = bound > tb ? count_hi(bound) : 65;
                if (few <= 64) {
                    compact([&](uint64_t v) __attribute__((always_inline)) { return (uint32_t)(v >> 32) >= bound; });
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    const uint64_t key = lane < few ? s_key[wave][lane] : 0ull;
                    const uint32_t hi = (uint32_t)(key >> 32);
                    const uint32_t cut = below(search_by(K, exact, [&](uint32_t v) __attribute__((always_inline)) { return __popcll(__ballot(hi >= v)); }));
                    // What was left out is below this.  (With K keys above the bound the search ends at the first prefix that all of them
                    // reach, which may lie below the bound and so below keys that are not here.  As a scalar: kept in a vector register, small fp32
                    // builds take 2 to 4 % longer, 2,000 x 320, K = 24: 61.3 us, 63.1.)
                    thr = (uint32_t)__builtin_amdgcn_readfirstlane((int)(cut > bound ? cut : bound));
                    const uint64_t m = __ballot(hi >= thr);
                    asm volatile("" ::: "memory");
                    if (hi >= thr) s_key[wave][__popcll(m & ((1ull << lane) - 1ull))] = key;
                    kept = __popcll(m);
                    return;
                }
            }
            uint32_t cut = below(search(K, exact));
            if (cut > tb) {
                kept = count_hi(cut);
                t = (uint64_t)cut << 32;
                thr = cut; // what was left out is below this
            }
            if (kept > KP * 64) {
                cut = search(KP * 64, exact);
                t = (uint64_t)cut << 32;
                if (!exact) { // keys of equal value straddle the cut: the ids (the lower half of the keys) decide
                    auto count_lo = [&](uint32_t v) __attribute__((always_inline)) {
                        int k = 0;
#pragma unroll
                        for (int r = 0; r < E; ++r)
                            if (E <= 8 || r * 64 < n) k += __popcll(__ballot((uint32_t)(val[r] >> 32) == cut && (uint32_t)val[r] >= v));
                        return k;
                    };
                    const int need = KP * 64 - (cut == 0xFFFFFFFFu ? 0 : count_hi(cut + 1u));
                    uint32_t t_lo = 0;
                    for (int bit = 31; bit >= 0; --bit) {
                        const uint32_t v = t_lo | (1u << bit);
                        if (count_lo(v) >= need) t_lo = v;
                    }
                    t |= t_lo;
                }
                thr = cut; // what was left out is at or below this
                kept = KP * 64;
            }
        }
        compact([&](uint64_t v) __attribute__((always_inline)) { return v >= t; }); // (kept of them)
    };
    if (SHORT && K <= 24 && n <= 256) select(std::integral_constant<int, 4>());
    else if (n <= 512) select(std::integral_constant<int, 8>());
    else select(std::integral_constant<int, GR_MAX_CAND / 64>());
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the keys written by the other lanes are in LDS
    if (overflow) thr = 0xFFFFFFFFu; // nothing is known about what was left out

    constexpr int S = KP + (HOP ? 1 : 0); // the last slot of a hop holds the list so far (K <= 64)
    double s[S];
    int32_t id[S];
#pragma unroll
    for (int t = 0; t < KP; ++t) {
        const int q = t * 64 + lane;
        s[t] = -INFINITY;
        id[t] = GR_NO_ID;
        if (q < kept) {
            const uint32_t j = 0xFFFFFFFFu - (uint32_t)s_key[wave][q];
            if (j < (uint64_t)Cv) { // always true for keys written by the recall pass
                id[t] = (int32_t)(visit_offset + j);
                s[t] = gr_canon(Wl + i * D, Wv + (int64_t)j * D, D);
            }
        }
    }
    if (HOP) {
        s[KP] = -INFINITY;
        id[KP] = GR_NO_ID;
        if (lane < K) {
            const int32_t g = graph[i * K + lane];
            if (g >= 0) {
                id[KP] = g;
                s[KP] = ((const double *)sims_)[i * K + lane];
            }
        }
        // a visiting row that is in the list already (a shard seen twice) is not a new candidate
        for (int src = 0; src < K; ++src) {
            const int32_t oid = __builtin_amdgcn_readlane(id[S - 1], src);
            if (oid == GR_NO_ID) continue;
#pragma unroll
            for (int t = 0; t < KP; ++t)
                if (id[t] == oid) {
                    id[t] = GR_NO_ID;
                    s[t] = -INFINITY;
                }
        }
    }
    // (entries without an id have similarity -inf and the largest id: they rank behind every real one)
    int rank[S];
#pragma unroll
    for (int t = 0; t < S; ++t) rank[t] = 0;
    int n_valid = 0;
#pragma unroll
    for (int t = 0; t < KP; ++t) {
        const int here = kept - t * 64 < 64 ? kept - t * 64 : 64;
        gr_count_before<S>(s[t], id[t], here, s, id, rank);
        n_valid += __popcll(__ballot(id[t] != GR_NO_ID));
    }
    if (HOP) {
        gr_count_before<S>(s[S - 1], id[S - 1], K, s, id, rank);
        n_valid += __popcll(__ballot(id[S - 1] != GR_NO_ID));
    }
    bool certified = true;
#pragma unroll
    for (int t = 0; t < S; ++t) {
        if (id[t] != GR_NO_ID && rank[t] < K) {
            graph[i * K + rank[t]] = id[t];
            if (HOP) ((double *)sims_)[i * K + rank[t]] = s[t];
            else if (sims_) ((float *)sims_)[i * K + rank[t]] = (float)s[t];
            if (rank[t] == K - 1) { // certificate: nothing that was dropped can reach the K-th exact similarity
                certified = s[t] > (double)gr_unorder(thr) + eps;
            }
        }
    }
    // A threshold of -infinity dropped nothing (a sample of fewer rows than its rank: every row passed).
    if (thr == gr_orderable(-INFINITY)) certified = true;
    else if (n_valid < K) certified = false; // no K-th candidate to certify
    if (HOP) {
        for (int e = n_valid + lane; e < K; e += 64) { // fewer than K known so far: empty slots
            graph[i * K + e] = -1;
            ((double *)sims_)[i * K + e] = -INFINITY;
        }
    } else if (n_valid < K) {
        certified = false;
    }
    if (__ballot(!certified) != 0ull && lane == 0) list_rows[atomicAdd(list_count, 1)] = (int32_t)i;
}

// ------------------------------------------------------------------------------------------------
// the same for the passes with running thresholds (K > 64 or D > 512), whose candidates are cut to k' <= 256 already
// ------------------------------------------------------------------------------------------------
template <typename IN>
__global__ void __launch_bounds__(GR_NT)
gr_rerank_kernel(const IN *__restrict__ W, int64_t C, int D, int K, int cap, const uint64_t *__restrict__ cand,
                 const int32_t *__restrict__ cnt, const uint32_t *__restrict__ thr, const float *__restrict__ norms,
                 const float *__restrict__ maxnorm, float gamma, int32_t *__restrict__ graph,
                 float *__restrict__ sims, int32_t *fb_count, int32_t *__restrict__ fb_rows) {
    const int64_t i = (int64_t)blockIdx.x * (GR_NT / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (i >= C) return;
    const int lane = threadIdx.x & 63;
    const int n = cnt[i];
    if (n < K && lane == 0) fb_rows[atomicAdd(fb_count, 1)] = (int32_t)i; // no K-th candidate to certify
    double s[4];
    int32_t id[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int q = t * 64 + lane;
        s[t] = -INFINITY;
        id[t] = GR_NO_ID;
        if (q < n) {
            const uint32_t j = 0xFFFFFFFFu - (uint32_t)cand[i * cap + q];
            if (j < (uint32_t)C) { // always true for keys written by the recall pass
                id[t] = (int32_t)j;
                s[t] = gr_canon(W + i * D, W + (int64_t)j * D, D);
            }
        }
    }
    int rank[4] = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < 4; ++t) gr_count_before<4>(s[t], id[t], n - t * 64 < 64 ? n - t * 64 : 64, s, id, rank);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int q = t * 64 + lane;
        if (q < n && rank[t] < K) {
            graph[i * K + rank[t]] = id[t];
            if (sims) sims[i * K + rank[t]] = (float)s[t];
            if (rank[t] == K - 1) {
                // certificate: nothing that was dropped can reach the K-th exact similarity
                const uint32_t th = thr[i];
                bool certified = (th == 0u); // nothing was ever dropped
                if (!certified) {
                    const double eps = (double)gamma * (double)norms[i] * (double)*maxnorm;
                    certified = s[t] > (double)gr_unorder(th) + eps;
                }
                if (!certified) fb_rows[atomicAdd(fb_count, 1)] = (int32_t)i;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// exhaustive fp64 search for the rows on the list
// ------------------------------------------------------------------------------------------------
template <typename IN>
__global__ void __launch_bounds__(GR_NT)
gr_exhaustive_kernel(const IN *__restrict__ W, int64_t C, int D, int K, const int32_t *__restrict__ fb_count,
                     const int32_t *__restrict__ fb_rows, double *__restrict__ scratch, int32_t *__restrict__ graph,
                     float *__restrict__ sims) {
    __shared__ double red_s[GR_NT];
    __shared__ int32_t red_j[GR_NT];
    __shared__ __attribute__((aligned(16))) IN row_i[GR_MAX_D];
    int n_fb = *fb_count;
    if (n_fb > C) n_fb = (int)C;
    double *my = scratch + (int64_t)blockIdx.x * C;
    for (int e = blockIdx.x; e < n_fb; e += gridDim.x) {
        const int64_t i = fb_rows[e];
        for (int d = threadIdx.x; d < D; d += GR_NT) row_i[d] = W[i * D + d];
        __syncthreads();
        for (int64_t j = threadIdx.x; j < C; j += GR_NT) my[j] = gr_canon(row_i, W + j * D, D);
        __syncthreads();
        double prev_s = INFINITY;
        int32_t prev_j = -1;
        for (int r = 0; r < K; ++r) {
            double best_s = -INFINITY;
            int32_t best_j = 0x7FFFFFFF;
            for (int64_t j = threadIdx.x; j < C; j += GR_NT) {
                if (j == i) continue;
                const double sj = my[j];
                if (gr_ranks_before(prev_s, prev_j, sj, (int32_t)j) && gr_ranks_before(sj, (int32_t)j, best_s, best_j)) {
                    best_s = sj;
                    best_j = (int32_t)j;
                }
            }
            red_s[threadIdx.x] = best_s;
            red_j[threadIdx.x] = best_j;
            __syncthreads();
            for (int o = GR_NT / 2; o > 0; o >>= 1) {
                if (threadIdx.x < o) {
                    if (gr_ranks_before(red_s[threadIdx.x + o], red_j[threadIdx.x + o], red_s[threadIdx.x], red_j[threadIdx.x])) {
                        red_s[threadIdx.x] = red_s[threadIdx.x + o];
                        red_j[threadIdx.x] = red_j[threadIdx.x + o];
                    }
                }
                __syncthreads();
            }
            prev_s = red_s[0];
            prev_j = red_j[0];
            if (threadIdx.x == 0) {
                graph[i * K + r] = prev_j;
                if (sims) sims[i * K + r] = (float)prev_s;
            }
            __syncthreads();
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Second chance for rows that the ranking of the k' best could not certify: the segments hold ALL rows above the row's
// fixed threshold (some 400), so the row is ranked again over all of them, and the certificate is taken against the fixed
// threshold, which lies far below the K-th neighbour.  It is what keeps tight clusters cheap: with hundreds of neighbours
// 2e-6 apart no k' of a few dozen spans the error bound, and the exhaustive search costs such a row 30 ms.  One wavefront
// per row; rows that still fail (a segment overflowed; ties at the fixed threshold) go to the exhaustive list.
// ------------------------------------------------------------------------------------------------
template <typename IN>
__global__ void __launch_bounds__(GR_NT)
gr_second_kernel(const IN *__restrict__ W, int64_t C, int D, int K, GrSegs seg, const uint64_t *__restrict__ cand,
                 const int32_t *__restrict__ cnt_res, const int32_t *__restrict__ cnt_str, const uint32_t *__restrict__ tbits,
                 const float *__restrict__ norms, const float *__restrict__ maxnorm, float gamma,
                 const int32_t *__restrict__ list_count, const int32_t *__restrict__ list_rows, int32_t *__restrict__ graph,
                 float *__restrict__ sims, int32_t *fb_count, int32_t *__restrict__ fb_rows) {
    __shared__ double s_s[GR_NT / 64][GR_MAX_CAND];
    __shared__ int32_t s_id[GR_NT / 64][GR_MAX_CAND];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nseg = 2 * seg.parts + (seg.stream > 0 ? 1 : 0);
    int64_t n_list = *list_count;
    if (n_list > C) n_list = C;
    for (int64_t e0 = (int64_t)blockIdx.x * (GR_NT / 64); e0 < n_list; e0 += (int64_t)gridDim.x * (GR_NT / 64)) {
        const int64_t e = e0 + wave;
        const int64_t i = e < n_list ? list_rows[e] : -1;
        int c_seg = 0, begin_seg = 0, n = 0, n_valid = 0;
        // (an overflowed segment does not hold everything above the threshold)
        bool usable = i >= 0 && !gr_segments(seg, cnt_res, cnt_str, i, c_seg, begin_seg);
        for (int sg = 0; sg < nseg && usable; ++sg) {
            const int c = __builtin_amdgcn_readlane(c_seg, sg), begin = __builtin_amdgcn_readlane(begin_seg, sg);
            if (n + c > GR_MAX_CAND) {
                usable = false;
                break;
            }
            for (int q = lane; q < c; q += 64) {
                double sv = -INFINITY;
                int32_t id = GR_NO_ID;
                const uint32_t j = 0xFFFFFFFFu - (uint32_t)cand[i * seg.cap() + begin + q];
                if (j < (uint32_t)C && (int64_t)j != i) { // always true for keys written by the recall pass
                    id = (int32_t)j;
                    sv = gr_canon(W + i * D, W + (int64_t)j * D, D);
                    ++n_valid;
                }
                s_s[wave][n + q] = sv;
                s_id[wave][n + q] = id;
            }
            n += c;
        }
        n_valid = ks_wave_sum_i(n_valid);
        __syncthreads();
        bool certified = usable && n_valid >= K;
        if (certified) {
            for (int q = lane; q < n; q += 64) {
                const double sv = s_s[wave][q];
                const int32_t id = s_id[wave][q];
                if (id == GR_NO_ID) continue;
                int rank = 0;
                for (int p = 0; p < n && rank < K; ++p) rank += gr_ranks_before(s_s[wave][p], s_id[wave][p], sv, id) ? 1 : 0;
                if (rank < K) {
                    graph[i * K + rank] = id;
                    if (sims) sims[i * K + rank] = (float)sv;
                    if (rank == K - 1) {
                        const double eps = (double)gamma * (double)norms[i] * (double)*maxnorm;
                        if (!(sv > (double)gr_unorder(tbits[i]) + eps)) certified = false;
                    }
                }
            }
        }
        if (i >= 0 && __ballot(!certified) != 0ull && lane == 0) fb_rows[atomicAdd(fb_count, 1)] = (int32_t)i;
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
static unsigned gr_sym_shares(int64_t C) { return (unsigned)ks_ceil_div(C, 256); } // a share per block of resident rows
static int gr_sym_chunks_stride(int64_t C, int D) { // chunks of a share at most: half of all groups, half of its own, a spare
    const int64_t nsb = ks_ceil_div(C, GR_SYM_SB), GS = gr_sym_group_sbs(C), NG = ks_ceil_div(nsb, GS);
    return (int)(((NG / 2) * GS + GS / 2 + 2) * (GR_SYM_SB / gr_chunk(D)));
}
// Fixed thresholds serve K <= 64 (a row with few candidates keeps them all and is certified against its fixed threshold).
// The resident rows' fragments of a depth beyond
// 512 do not fit in registers.  A row id has 22 bits in the stream side's records; beyond them (and for lists that no
// device memory holds twice) the running thresholds stay.
static bool gr_use_fixed(int64_t Cr, int64_t Cs, int D, int K) {
    return K <= 64 && D <= 512 && Cr <= ((int64_t)1 << 22) && Cs <= ((int64_t)1 << 22);
}
// The division of the symmetric sweep exists from 6,144 rows on; it is used from C * D = 11 million on, at D = 128 from 15 million.
// Below, the passes over both halves of the pairs (gr_recall_fix_kernel) are faster: the matrix cores idle anyway, and what
// costs is the epilogue's work per hit, of which the stream side's is the dearer one.  Whole builds of bf16 rows, us, parts -> symmetric:
// D = 512: 12,000, K = 8: 238, 259; 15,000, K = 32: 358, 387; 18,000: K = 16 447, 426, K = 64 573, 596; 21,500: K = 8 573, 491, K = 32 593, 539, K =
// 64 717, 686; 26,000: K = 8 814, 633, K = 64 992, 864.  D = 256: 22,000, K = 16: 392, 408; 34,000: K = 8 773, 702, K = 64 928, 957; 43,000: K = 8
// 1,094, 908, K = 32 1,142, 1,034, K = 64 1,277, 1,226; 52,000: K = 16 1,586, 1,315, K = 64 1,787, 1,723.
// At D = 128 neither is the faster one on one side of a size: the parts' time goes up in steps of 256 blocks (65,536 and 131,072 rows),
// the symmetric pass has steps of its own, and where one row in 32 is sampled (K > 24, fp32) its records cost more.  72,000: K = 16 2,099,
// 2,073, K = 64 2,355, 2,460; 86,000: K = 16 2,748, 2,777, K = 32 2,795, 3,009; 100,000: K = 16 3,804, 3,531, K = 32 3,884, 3,780; 105,000, K = 32:
// 4,157, 4,390; 115,000: K = 16 5,216, 5,013, K = 32 5,308, 5,768; 117,500: K = 16 5,335, 5,049, K = 32 5,448, 5,765; 126,000: K = 16 5,740, 5,493,
// K = 32 5,840, 6,260, K = 64 6,152, 6,784; 136,000: K = 16 7,376, 6,727, K = 32 7,545, 7,043; 150,000, K = 32: 7,851, 7,713.  So from 15 million on the
// symmetric pass is right for K <= 24, and for larger K (and fp32) only from 16.8 million, 131,072 rows, on: between the two lines they
// take 4 to 18 % longer than in parts, and less than before the sweep in turns all the same.
static bool gr_has_sym(int64_t C, int D, int K) {
    return (D == 128 || D == 256 || D == 512) && gr_use_fixed(C, C, D, K) && C >= 6144;
}
static bool gr_use_sym(int64_t C, int D, int K) { return gr_has_sym(C, D, K) && C * D >= (D == 128 ? 15000000 : 11000000); }
// Parts that the streamed chunks of each of nb blocks are cut into: the number with the least estimated time on the
// chip's compute units (rounds of workgroups x (set-up + chunks of a part); set-up 6 us and a chunk of 96 rows 1.2 us,
// 0.5 and 0.4 us more per k-tile: measured on the plain sweep).  Bounded by memory: a part costs every row two segments.
static int gr_parts(int64_t C, int64_t nb, int64_t chunks, int D) {
    const double kt = (D + 63) / 64, setup = 6.0 + 0.5 * kt, per_chunk = 1.2 + 0.4 * kt;
    int64_t most = ((int64_t)1 << 19) / C; // 4.5 to 5.5 GiB of segments
    if (most > GR_MAX_PARTS) most = GR_MAX_PARTS;
    if (most > chunks) most = chunks;
    int best = 1;
    double best_t = 0.0;
    for (int p = 1; p <= most || p == 1; ++p) {
        const double t = (double)ks_ceil_div(nb * p, GR_CUS) * (setup + (double)ks_ceil_div(chunks, p) * per_chunk);
        if (p == 1 || t < 0.98 * best_t) { best = p; best_t = t; }
    }
    return best;
}

// Searched rows per sampled row, and the place in the sorted list.  A hit costs the recall and the ranking the same whatever
// the problem's size, a sampled row costs a product per row: the denser sample pays in smaller problems.  One in 16 (place 8, 10,
// 12 for K <= 8, 16, 24: 128, 160, 192 candidates instead of 256, 256, 320), us, 32 -> 16: 10,000 x 128, K = 8: 119 -> 106;
// 20,000 x 64, K = 16: 248 -> 225; 60,000 x 256, K = 16: 2,402 -> 2,242; 130,000 x 128, K = 24: 6,646 -> 6,199; 300,000 x 128,
// K = 16: 30,532 -> 29,495, hence C * D <= 50 million.  Deeper than 256 a sampled row costs more and it pays up to 15 million
// (30,000 x 512, K = 16: 969 -> 962; 45,000 x 320, K = 8: 1,679 -> 1,678; but 48,000 x 512, K = 16: 1,813 -> 1,818; 100,000 x 320,
// K = 16: 7,518 -> 7,650; 90,000 x 512, K = 16: 5,854 -> 5,977), at D = 512 with K > 16, the symmetric sweep and 128 fewer
// candidates, up to 30 million (58,000, K = 24: 2,738 -> 2,659; but 70,000: 4,187 -> 4,204).  Without that sweep and
// with K > 8 it pays up to 96,000 rows (95,000 x 64, K = 16: 2,463 -> 2,439; 90,000 x 128: 3,425 -> 3,416; x 192: 4,367 -> 4,352;
// but 110,000 x 64: 3,020 -> 3,064; x 128: 4,928 -> 4,986; x 192: 6,371 -> 6,454; 180,000 x 192: 16,860 -> 17,067; with K = 8 still
// 4,914 -> 4,883 at 110,000 x 128 and 16,797 -> 16,752 at 180,000 x 192), at 96 throughout (195,000, K = 16: 12,754 -> 12,696).
// fp32 rows stay: their error bound is that of rounding the rows to bf16, and with a threshold closer to the K-th neighbour
// more rows of tight clusters have no certificate (20,000 x 256 in clusters of 200 with noise of 0.1: 36 -> 290 ms).  So does
// K > 24: with 12 places two rows in a million find at most 32 (a tenth of that as it is), and one such row in the exhaustive
// pass costs more than the sample gives (120,000 x 64, K = 32: 3,921 -> 5,298).  A hop's lists give better thresholds than a
// denser sample after the first one (2,000 x 2,000 x 256 with full lists: 42 -> 44): it stays too.
// The chance that a row finds at most K is one in ten million at K = 24.
static int gr_every(int64_t C, int D, int K, int dtype, bool hop) {
    int64_t most = D <= 256 ? 50000000 : (D == 512 && K > 16 ? 30000000 : 15000000);
    if (!gr_use_sym(C, D, K) && K > 8 && (D == 64 || D >= 128) && C > 96000) most = 0;
    return !hop && dtype == KS_DTYPE_BF16 && K <= 24 && C * D <= most ? 16 : 32;
}
static int gr_rank_of(int K, int every) {
    if (every == 16) return K <= 8 ? 8 : (K <= 16 ? 10 : 12);
    return K <= 16 ? 8 : (K <= 32 ? 10 : GR_RANK);
}
// Workgroups per block of resident rows for the sample: the number with the least estimated time (rounds of workgroups x
// (set-up + chunks), as in gr_parts, a chunk's insertions 1.5 us more; merging the lists in the recall pass 4 us and 0.3 per list).
// 10,000 x 128: 40 blocks of 4 chunks, 19.8 -> 11.2 us with four; 25,000 x 256: 98 of 9, 47 -> 32 with two.
// The sampled rows and their lists are done with when the ranking starts and lie in the exhaustive pass's scratch, 512 bytes per
// searched row: 64 at most for the rows, 48 per part and resident row for the lists.  A hop of many rows over few has parts only
// as far as that goes.
static_assert(GR_FB_BLOCKS * sizeof(double) >= 2 * 512 / 16 + GR_SAMPLE_PARTS * GR_RANK * sizeof(float), "a build has room for all parts");
static GrSample gr_sample_plan(int64_t Cr, int64_t Cs, int every, int D, int r, bool sym) {
    const int64_t n_sample = Cs / every;
    const size_t room = (size_t)GR_FB_BLOCKS * Cs * sizeof(double), rows = ks_align_up((size_t)n_sample * D * sizeof(uint16_t), 256);
    const int64_t nb = ks_ceil_div(Cr, 256), chunks = ks_ceil_div(n_sample, 96);
    const double kt = (D + 63) / 64, setup = 6.0 + 0.5 * kt, per_chunk = 2.7 + 0.4 * kt;
    int best = 1;
    double best_t = 0.0;
    for (int p = 1; p == 1 || (p <= chunks && p <= GR_SAMPLE_PARTS && !sym); ++p) { // (the symmetric sweep wants the thresholds ready)
        if (p > 1 && rows + (size_t)p * GR_RANK * Cr * sizeof(float) > room) break;
        const double t = (double)ks_ceil_div(nb * p, GR_CUS) * (setup + (double)ks_ceil_div(chunks, p) * per_chunk) + (p > 1 ? 4.0 + 0.3 * p : 0.0);
        if (p == 1 || t < 0.98 * best_t) { best = p; best_t = t; }
    }
    GrSample smp;
    smp.r = r;
    smp.part_rows = (int)(ks_ceil_div(chunks, best) * 96);
    smp.parts = chunks > 0 ? (int)ks_ceil_div(n_sample, smp.part_rows) : 1; // (rounding up may leave the last without rows)
    smp.tops = nullptr;
    return smp;
}

// how a pass with fixed thresholds divides its work and a row's segments
struct GrFixPlan {
    GrSegs seg;
    int room_parts, room; // what a row has room for in the workspace: parts, slots
    bool turns;           // parts: sweep in turns
    int part_rows;        // streamed rows per part (not the symmetric sweep)
    int log_rows, logs;   // symmetric sweep: rows per log, number of logs
    int every;            // searched rows per sampled row
    GrSample smp;
};
static GrFixPlan gr_fix_plan(int64_t Cr, int64_t Cs, int D, int K, int dtype, bool sym, bool hop) {
    GrFixPlan f;
    f.every = gr_every(Cs, D, K, dtype, hop);
    f.smp = gr_sample_plan(Cr, Cs, f.every, D, gr_rank_of(K, f.every), sym);
    const int64_t nb = ks_ceil_div(Cr, 256), ch = gr_chunk(D), chunks = ks_ceil_div(Cs, 96);
    f.seg.parts = gr_parts(Cr, nb, sym ? chunks / 2 + 8 : chunks, D);
    const int q_most = sym ? GR_SYM_Q : 32 * (gr_rank_of(K, 32) + 10) + 24; // (with the denser sample: room for ties)
    f.seg.q = q_most;
    f.seg.stream = sym ? GR_SYM_SCAP : 0;
    f.part_rows = (int)(ks_ceil_div(chunks, f.seg.parts) * 96);
    f.room_parts = sym ? f.seg.parts : (int)ks_ceil_div(Cs, f.part_rows); // (rounding up may leave the last parts without rows)
    f.turns = false;
    if (!sym && f.seg.q > f.part_rows / 2) f.seg.q = f.part_rows / 2;
    f.room = 2 * f.room_parts * f.seg.q + f.seg.stream;
    if (!sym) {
        // The room is planned in chunks of 96 rows whatever the sweep's are: a workspace serves what it always did.  The parts are whole
        // chunks of the sweep where those fit in it; otherwise (builds of up to 12,000 rows, hops of few rows to 35,000 visiting ones) the last
        // chunk of each is a ragged one.
        // In turns from seven chunks of 96 rows on: with fewer there is little to take turns in, and larger chunks fit the parts less
        // well (2,000 x 64, one chunk a part: 41.5 us, in turns 42.4; 2,345 x 128: 58.2, 59.8; 5,500 x 256, six: 76.5, 77.1; 8,000 x
        // 320, eleven: 129.5, 119.2; 10,000 x 128: 124.0, 119.2).
        f.seg.parts = f.room_parts;
        // At D = 32 and 64 a compute unit has room for two workgroups of the plain sweep (120 registers, 72 KiB of LDS; in turns 214), which
        // cover each other's epilogues better than two halves do: there in turns only where no two workgroups meet.  Plain, in turns:
        // x 64, K = 32: 20,000 (237 workgroups) 253 us, 238; 26,000 280, 339; 50,000 780, 953; 150,000 5,170, 6,914; x 32, K = 8: 20,000 201,
        // 189; 50,000 649, 868; 150,000 4,264, 5,930; a hop of 50,000 x 20,000 x 64, K = 16: 444, 533.
        f.turns = f.part_rows >= 672 && (D > 64 || nb * f.room_parts <= GR_CUS);
        const int rows = (int)(ks_ceil_div(ks_ceil_div(Cs, ch), f.room_parts) * ch), parts = (int)ks_ceil_div(Cs, rows);
        const int64_t half = ((rows < Cs ? rows : Cs) + 1) / 2; // (in turns some 300 at least: a lane looks for room for a block's 16 hits)
        const int q = half < q_most ? (int)half : q_most;
        if (f.turns && 2 * parts * q <= f.room) { f.part_rows = rows; f.seg.parts = parts; f.seg.q = q; }
    }
    f.log_rows = GR_SYM_SB;
    f.logs = 0;
    if (sym) {
        // A wavefront finds about 32 * 384 / C stream-side hits per streamed row.  Logs of half a super-block where its 384 rows (six
        // chunks at D = 512, three at 128) still give it half a batch (C <= 49,152): the scatter kernel then has 77 workgroups or more
        // instead of 39.
        if ((double)(GR_SYM_SB / 2) * 32.0 * 384.0 / (double)Cs >= 96.0) f.log_rows = GR_SYM_SB / 2;
        f.logs = (int)ks_ceil_div(Cr, f.log_rows);
    }
    return f;
}

struct GrWs {
    uint16_t *Wb;
    float *norms, *blockmax, *maxnorm;
    uint64_t *cand;
    int32_t *fb_count;
    int32_t *fb_rows;
    double *scratch;
    // running thresholds
    int32_t *cnt;
    uint32_t *thr;
    // fixed thresholds
    uint16_t *Ws;      // sampled rows
    float *tops, *thf;
    uint32_t *tbits;
    int32_t *cnt_res, *cnt_str;
    int32_t *second_count, *second_rows; // rows for gr_second_kernel
    // every similarity computed once
    int32_t *logcnt, *plan;
    int2 *chunks;
    uint2 *log;
};

static GrWs gr_carve(void *ws, int64_t C, int D, int K, int dtype, size_t *total) {
    KsArena ar(ws);
    GrParams p = gr_params(K, D);
    const bool fixed = gr_use_fixed(C, C, D, K), sym = gr_use_sym(C, D, K);
    GrWs w = GrWs();
    w.Wb = dtype == KS_DTYPE_FP32 ? ar.take<uint16_t>((size_t)C * D) : nullptr;
    w.norms = ar.take<float>((size_t)C);
    w.blockmax = ar.take<float>(GR_PREP_BLOCKS);
    w.maxnorm = ar.take<float>(1);
    w.fb_count = ar.take<int32_t>(1);
    w.fb_rows = ar.take<int32_t>((size_t)C);
    w.scratch = ar.take<double>((size_t)GR_FB_BLOCKS * C);
    if (!fixed) {
        w.cand = ar.take<uint64_t>((size_t)C * p.cap);
        w.cnt = ar.take<int32_t>((size_t)C);
        w.thr = ar.take<uint32_t>((size_t)C);
    } else {
        const GrFixPlan f = gr_fix_plan(C, C, D, K, dtype, sym, false);
        const int64_t Cpad = ks_ceil_div(C, GR_SYM_SB) * GR_SYM_SB + 128;
        w.cand = ar.take<uint64_t>((size_t)C * f.room);
        KsArena over(w.scratch); // see gr_sample_plan
        w.Ws = over.take<uint16_t>((size_t)(C / f.every) * D);
        w.tops = f.smp.parts > 1 ? over.take<float>((size_t)f.smp.parts * GR_RANK * C) : nullptr;
        w.thf = ar.take<float>((size_t)Cpad);
        w.tbits = ar.take<uint32_t>((size_t)C);
        w.cnt_res = ar.take<int32_t>((size_t)C * 2 * f.room_parts);
        w.second_count = ar.take<int32_t>(1);
        w.second_rows = ar.take<int32_t>((size_t)C);
        if (sym) {
            w.cnt_str = ar.take<int32_t>((size_t)C);
            w.logcnt = ar.take<int32_t>((size_t)f.logs);
            w.plan = ar.take<int32_t>((size_t)gr_sym_shares(C) * GR_SYM_PLAN);
            w.chunks = ar.take<int2>((size_t)gr_sym_shares(C) * gr_sym_chunks_stride(C, D));
            w.log = ar.take<uint2>((size_t)f.logs * f.log_rows * GR_SYM_LOG_PER_ROW);
        }
    }
    if (total) *total = ar.off;
    return w;
}

static int gr_check(int64_t C, int D, int K, int dtype) {
    if (dtype != KS_DTYPE_BF16 && dtype != KS_DTYPE_FP32) return KS_INVALID_ARG;
    if (C < 2 || C >= (int64_t)1 << 31 || D < 32 || D % 32 != 0 || K < 1) return KS_INVALID_ARG;
    if (K > KS_MAX_GRAPH_K || K > C - 1 || D > GR_MAX_D) return KS_UNSUPPORTED;
    return KS_OK;
}

extern "C" int knn_graph_build_plan(int64_t C, int D, int K, int dtype, int workgroup, int32_t *n_workgroups, int32_t *out) {
    if (!n_workgroups) return KS_INVALID_ARG;
    int rc = gr_check(C, D, K, dtype);
    if (rc != KS_OK) return rc;
    *n_workgroups = 0;
    if (!gr_has_sym(C, D, K)) return KS_OK;
    *n_workgroups = (int32_t)gr_sym_shares(C);
    if (!out) return KS_OK;
    if (workgroup < 0 || workgroup >= *n_workgroups) return KS_INVALID_ARG;
    const GrSymRanges r = gr_sym_ranges(workgroup, (int)C, gr_sym_group_sbs(C));
    out[0] = r.block;
    for (int part = 0; part < 5; ++part) { out[1 + 2 * part] = r.first[part]; out[2 + 2 * part] = r.end[part]; }
    // which of the (up to three) 256-row blocks of its own super-block it pairs with: bit k = block k of that super-block
    int mask = 0;
    if (r.block >= 0) {
        const int kb = r.ring & 15, n_b = (r.ring >> 4) & 15, succ_b = r.ring >> 8;
        for (int k = 0; k < n_b; ++k) {
            const int dd = (k - kb + n_b) % n_b;
            if (dd >= 1 && dd <= succ_b) mask |= 1 << k;
        }
    }
    out[11] = mask;
    return KS_OK;
}

extern "C" size_t knn_graph_build_workspace(int64_t C, int D, int K, int dtype) {
    if (gr_check(C, D, K, dtype) != KS_OK) return 0;
    size_t total = 0;
    gr_carve(nullptr, C, D, K, dtype, &total);
    return total;
}

static GrPrepJob gr_prep_job(const void *W, int64_t C, int D, int dtype, uint16_t *Wb, float *norms, float *blockmax, uint16_t *Ws, int every) {
    GrPrepJob j;
    j.every = every;
    j.W = W;
    j.C = C;
    j.Wb = Wb;
    j.norms = norms;
    j.blockmax = blockmax;
    j.Ws = Ws;
    j.n_sample = Ws ? C / every : 0;
    // four row groups per wavefront: a wavefront takes 64 / (lanes per row) rows at a time
    const int pieces = D * (dtype == KS_DTYPE_BF16 ? 2 : 4) / 16;
    int64_t rows = 64 / (pieces > 32 ? 64 : (pieces > 16 ? 32 : (pieces > 8 ? 16 : (pieces > 4 ? 8 : 4)))) * (GR_NT / 64) * 2;
    const int64_t b = ks_ceil_div(C, rows);
    j.blocks = (int)(b < GR_PREP_BLOCKS ? b : GR_PREP_BLOCKS);
    return j;
}
static void gr_launch_prepare(const GrPrepJob &j0, const GrPrepJob &j1, int D, int dtype, const GrClear &clr, hipStream_t st) {
    const dim3 grid((unsigned)(j0.blocks + j1.blocks));
    if (dtype == KS_DTYPE_FP32) hipLaunchKernelGGL(gr_prepare_kernel<float>, grid, dim3(GR_NT), 0, st, j0, j1, D, clr);
    else hipLaunchKernelGGL(gr_prepare_kernel<uint16_t>, grid, dim3(GR_NT), 0, st, j0, j1, D, clr);
}

// Sweeps of a depth of KT k-tiles (D <= 512, D % 32 == 0): F(KT, RAGGED) is instantiated
#define GR_FOR_DEPTH(F)                                                                                     \
    do {                                                                                                    \
        const int kt = (D + 63) / 64;                                                                       \
        if (D % 64 == 0) {                                                                                  \
            if (kt == 1) F(1, false); else if (kt == 2) F(2, false); else if (kt == 3) F(3, false);         \
            else if (kt == 4) F(4, false); else if (kt == 5) F(5, false); else if (kt == 6) F(6, false);    \
            else if (kt == 7) F(7, false); else F(8, false);                                                \
        } else {                                                                                            \
            if (kt == 1) F(1, true); else if (kt == 2) F(2, true); else if (kt == 3) F(3, true);            \
            else if (kt == 4) F(4, true); else if (kt == 5) F(5, true); else if (kt == 6) F(6, true);       \
            else if (kt == 7) F(7, true); else F(8, true);                                                  \
        }                                                                                                   \
    } while (0)

static void gr_launch_threshold(const uint16_t *R, int64_t Cr, const uint16_t *Ws, int64_t n_sample, int D, const GrSample &smp, const float *blockmax,
                                int n_blockmax, float *maxnorm, const GrHop &hop, float *thf, uint32_t *tbits, hipStream_t st) {
    const dim3 grid((unsigned)(ks_ceil_div(Cr, 256) * smp.parts));
#define GR_THR_LAUNCH(KT, RAGGED)                                                                                                    \
    do {                                                                                                                      \
        if (smp.parts > 1)                                                                                                    \
            hipLaunchKernelGGL((gr_threshold_kernel<KT, RAGGED, true>), grid, dim3(512), 0, st, R, Cr, Ws, (int)n_sample, D, smp, blockmax, \
                               n_blockmax, maxnorm, hop, thf, tbits);                                                         \
        else                                                                                                                  \
            hipLaunchKernelGGL((gr_threshold_kernel<KT, RAGGED, false>), grid, dim3(512), 0, st, R, Cr, Ws, (int)n_sample, D, smp, blockmax, \
                               n_blockmax, maxnorm, hop, thf, tbits);                                                         \
    } while (0)
    GR_FOR_DEPTH(GR_THR_LAUNCH);
#undef GR_THR_LAUNCH
}
static void gr_launch_recall_fix(const GrPair &pr, int D, const GrFixPlan &f, const GrSample &smp, const GrHop &hop, const float *maxnorm,
                                 const float *thf, uint32_t *tbits, uint64_t *cand, int32_t *cnt_res, hipStream_t st) {
    const int nb = (int)ks_ceil_div(pr.Cr, 256);
    const dim3 grid((unsigned)(nb * f.seg.parts));
    const GrMerge merge{smp, hop, maxnorm, tbits};
#define GR_FIX_LAUNCH2(KT, RAGGED, TURNS)                                                                                             \
    do {                                                                                                                            \
        if (smp.parts > 1)                                                                                                          \
            hipLaunchKernelGGL((gr_recall_fix_kernel<KT, RAGGED, GrMerge, TURNS>), grid, dim3(512), 0, st, pr, D, nb, f.part_rows, f.seg, \
                               merge, thf, cand, cnt_res);                                                                          \
        else                                                                                                                        \
            hipLaunchKernelGGL((gr_recall_fix_kernel<KT, RAGGED, GrReady, TURNS>), grid, dim3(512), 0, st, pr, D, nb, f.part_rows, f.seg, \
                               GrReady(), thf, cand, cnt_res);                                                                      \
    } while (0)
#define GR_FIX_LAUNCH(KT, RAGGED)                          \
    do {                                                   \
        if (f.turns) GR_FIX_LAUNCH2(KT, RAGGED, true);     \
        else GR_FIX_LAUNCH2(KT, RAGGED, false);            \
    } while (0)
    GR_FOR_DEPTH(GR_FIX_LAUNCH);
#undef GR_FIX_LAUNCH
#undef GR_FIX_LAUNCH2
}

// thr_init (optional, honoured by the sweep kernel only, may be `thr`): per row the value bits of a similarity at or below
// which no candidate is wanted
static void gr_launch_recall(const GrPair &pr, int D, const GrParams &p, uint64_t *cand, int32_t *cnt, uint32_t *thr,
                             hipStream_t st, const uint32_t *thr_init = nullptr) {
    const int64_t C = pr.Cr;
    if (D == 128 || D == 256 || D == 512) {
        const unsigned nb = (unsigned)ks_ceil_div(C, 256);
#define GR_SOE_LAUNCH(KT)                                                                                                   \
    do {                                                                                                                    \
        if (p.cap == 256)                                                                                                   \
            hipLaunchKernelGGL((gr_recall_soe_kernel<KT, 4>), dim3(nb), dim3(512), 0, st, pr, D, p.kprime, cand, cnt, thr,  \
                               thr_init);                                                                                   \
        else                                                                                                                \
            hipLaunchKernelGGL((gr_recall_soe_kernel<KT, 8>), dim3(nb), dim3(512), 0, st, pr, D, p.kprime, cand, cnt, thr,  \
                               thr_init);                                                                                   \
    } while (0)
        if (D == 512) GR_SOE_LAUNCH(8);
        else if (D == 256) GR_SOE_LAUNCH(4);
        else GR_SOE_LAUNCH(2);
#undef GR_SOE_LAUNCH
    } else if (D % 64 == 0) {
        hipLaunchKernelGGL((gr_recall_async_kernel<TileRA, 8>), dim3((unsigned)ks_ceil_div(C, TileRA::BM)), dim3(TileRA::NT), 0,
                           st, pr, D, p.kprime, cand, cnt, thr);
    } else {
        const unsigned recall_blocks = (unsigned)ks_ceil_div(C, TileR::BM);
        if (p.cap == 256)
            hipLaunchKernelGGL((gr_recall_kernel<TileR, 4>), dim3(recall_blocks), dim3(TileR::NT), 0, st, pr, D, p.kprime, cand,
                               cnt, thr);
        else
            hipLaunchKernelGGL((gr_recall_kernel<TileR, 8>), dim3(recall_blocks), dim3(TileR::NT), 0, st, pr, D, p.kprime, cand,
                               cnt, thr);
    }
}

// W searched in W with every similarity computed once: the sweep, the stream side's records to their rows
static void gr_launch_recall_sym(const uint16_t *Wb, int64_t C, int D, const GrFixPlan &f, const GrWs &w, hipStream_t st) {
    const unsigned shares = gr_sym_shares(C), grid = shares * (unsigned)f.seg.parts;
    const int stride = gr_sym_chunks_stride(C, D);
    hipLaunchKernelGGL(gr_sym_plan_kernel, dim3(shares), dim3(GR_NT), 0, st, (int)C, gr_sym_group_sbs(C), gr_chunk(D), w.plan, w.chunks, stride);
    const bool split = f.seg.parts > 1 || f.log_rows != GR_SYM_SB;
#define GR_SYM_LAUNCH2(KT, SPLIT)                                                                                              \
    hipLaunchKernelGGL((gr_recall_sym_kernel<KT, SPLIT>), dim3(grid), dim3(512), 0, st, Wb, (int)C, D, w.plan, w.chunks, stride, \
                       f.seg.parts, f.log_rows, w.thf, w.cand, w.cnt_res, w.log, w.logcnt)
#define GR_SYM_LAUNCH(KT)                        \
    do {                                         \
        if (split) GR_SYM_LAUNCH2(KT, true);     \
        else GR_SYM_LAUNCH2(KT, false);          \
    } while (0)
    if (D == 512) GR_SYM_LAUNCH(8);
    else if (D == 256) GR_SYM_LAUNCH(4);
    else GR_SYM_LAUNCH(2);
#undef GR_SYM_LAUNCH
#undef GR_SYM_LAUNCH2
    hipLaunchKernelGGL(gr_sym_scatter_kernel, dim3((unsigned)f.logs), dim3(1024), 0, st, w.log, w.logcnt, (int)C, f.log_rows, f.seg,
                       w.cand, w.cnt_str);
}

// error bound of the recall pass relative to |w_i||w_j|: fp32 accumulation of D exact bf16 products
// (2^-23 per addition allows for truncating adders), plus the bf16 rounding of both rows (2 * 2^-9,
// rounded up to 2^-7.9) when the input is fp32; a small slack covers the fp32 norms themselves
static float gr_gamma(int D, int dtype) {
    float gamma = (float)D * 1.1920929e-7f * 1.01f;
    if (dtype == KS_DTYPE_FP32) gamma += 0.0042f;
    return gamma;
}

// ranking of the candidates, and the second chance of the rows that it could not certify
template <typename IN>
static void gr_launch_rank(const IN *W, int64_t C, int D, int K, const GrFixPlan &f, const GrWs &w, float gamma,
                           int32_t *graph, float *sims, hipStream_t st) {
    const dim3 grid((unsigned)ks_ceil_div(C, GR_NT / 64));
#define GR_RANK_LAUNCH(KP, SHORT, LANES)                                                                                       \
    hipLaunchKernelGGL((gr_rank_kernel<IN, KP, false, SHORT, LANES>), grid, dim3(GR_NT), 0, st, W, C, W, C, D, K, f.seg, w.cand,        \
                       w.cnt_res, w.cnt_str, w.tbits, w.norms, w.maxnorm, gamma, (int64_t)0, graph, (void *)sims, w.second_count, \
                       w.second_rows)
    if (K <= 24 && (sizeof(IN) == 2 || C > GR_RANK_AT_ONCE)) GR_RANK_LAUNCH(1, true, true);
    else if (K <= 29 || (K <= 32 && D <= 128)) GR_RANK_LAUNCH(1, false, true);
    else if (K <= 32) GR_RANK_LAUNCH(1, false, sizeof(IN) == 2);
    else if (sizeof(IN) == 2 && C > GR_RANK_AT_ONCE) GR_RANK_LAUNCH(2, true, false);
    else GR_RANK_LAUNCH(2, false, false);
#undef GR_RANK_LAUNCH
    // (as many workgroups as run at once, by their LDS: nearly always there is nothing to do, and four rounds of that take 1 to 2 us more)
    hipLaunchKernelGGL(gr_second_kernel<IN>, dim3(GR_CUS), dim3(GR_NT), 0, st, W, C, D, K, f.seg, w.cand, w.cnt_res, w.cnt_str, w.tbits,
                       w.norms, w.maxnorm, gamma, w.second_count, w.second_rows, graph, sims, w.fb_count, w.fb_rows);
}

extern "C" int knn_graph_build(const void *W, int dtype, int64_t C, int D, int K, int32_t *graph, float *sims, void *ws,
                               size_t ws_bytes, int32_t *dev_status, void *stream) {
    (void)dev_status;
    if (!W || !graph || !ws) return KS_INVALID_ARG;
    int rc = gr_check(C, D, K, dtype);
    if (rc != KS_OK) return rc;
    size_t need = 0;
    GrWs w = gr_carve(ws, C, D, K, dtype, &need);
    if (ws_bytes < need) return KS_WORKSPACE_TOO_SMALL;
    const GrParams p = gr_params(K, D, dtype);
    hipStream_t st = (hipStream_t)stream;
    const bool fixed = gr_use_fixed(C, C, D, K), sym = gr_use_sym(C, D, K);
    const GrFixPlan f = gr_fix_plan(C, C, D, K, dtype, sym, false);
    GrClear clr = GrClear();
    clr.fb_count = w.fb_count;
    if (fixed) clr.second_count = w.second_count;
    if (sym) {
        clr.logcnt = w.logcnt;
        clr.nlog = f.logs;
        clr.thf = w.thf;
        clr.pad0 = C;
        clr.pad1 = ks_ceil_div(C, GR_SYM_SB) * GR_SYM_SB + 128;
    }
    const GrPrepJob job = gr_prep_job(W, C, D, dtype, w.Wb, w.norms, w.blockmax, fixed ? w.Ws : nullptr, f.every);
    gr_launch_prepare(job, GrPrepJob(), D, dtype, clr, st);
    const uint16_t *Wb = dtype == KS_DTYPE_FP32 ? w.Wb : (const uint16_t *)W;
    const GrPair pr{Wb, C, Wb, C, 0};
    const float gamma = gr_gamma(D, dtype);
    if (fixed) {
        GrSample smp = f.smp;
        smp.tops = w.tops;
        gr_launch_threshold(Wb, C, w.Ws, job.n_sample, D, smp, w.blockmax, job.blocks, w.maxnorm, GrHop(), w.thf, w.tbits, st);
        if (sym) gr_launch_recall_sym(Wb, C, D, f, w, st);
        else gr_launch_recall_fix(pr, D, f, smp, GrHop(), w.maxnorm, w.thf, w.tbits, w.cand, w.cnt_res, st);
        if (dtype == KS_DTYPE_FP32) gr_launch_rank<float>((const float *)W, C, D, K, f, w, gamma, graph, sims, st);
        else gr_launch_rank<uint16_t>((const uint16_t *)W, C, D, K, f, w, gamma, graph, sims, st);
    } else {
        hipLaunchKernelGGL(gr_maxnorm_kernel, dim3(1), dim3(64), 0, st, w.blockmax, job.blocks, w.maxnorm);
        gr_launch_recall(pr, D, p, w.cand, w.cnt, w.thr, st);
        const dim3 grid((unsigned)ks_ceil_div(C, GR_NT / 64));
        if (dtype == KS_DTYPE_FP32)
            hipLaunchKernelGGL(gr_rerank_kernel<float>, grid, dim3(GR_NT), 0, st, (const float *)W, C, D, K, p.cap, w.cand, w.cnt, w.thr,
                               w.norms, w.maxnorm, gamma, graph, sims, w.fb_count, w.fb_rows);
        else
            hipLaunchKernelGGL(gr_rerank_kernel<uint16_t>, grid, dim3(GR_NT), 0, st, (const uint16_t *)W, C, D, K, p.cap, w.cand, w.cnt,
                               w.thr, w.norms, w.maxnorm, gamma, graph, sims, w.fb_count, w.fb_rows);
    }
    if (dtype == KS_DTYPE_FP32)
        hipLaunchKernelGGL(gr_exhaustive_kernel<float>, dim3(GR_FB_BLOCKS), dim3(GR_NT), 0, st, (const float *)W, C, D, K, w.fb_count,
                           w.fb_rows, w.scratch, graph, sims);
    else
        hipLaunchKernelGGL(gr_exhaustive_kernel<uint16_t>, dim3(GR_FB_BLOCKS), dim3(GR_NT), 0, st, (const uint16_t *)W, C, D, K,
                           w.fb_count, w.fb_rows, w.scratch, graph, sims);
    KS_LAUNCH_CHECK();
    return KS_OK;
}

// ------------------------------------------------------------------------------------------------
// One hop of the distributed graph build (Section 3.2.2: the shards of W travel from node to node, each node
// searches every visiting shard and keeps its rows' best K so far).  Recall pass of the node's rows against the
// visiting rows as above; then per row an exact merge of the recalled candidates with the list so far, on
// (canonical fp64 similarity descending, id of the whole problem ascending), with the same certificate; rows
// that fail it are merged against every visiting row.
// ------------------------------------------------------------------------------------------------
// Running thresholds (K > 64 or D > 512): one wavefront per row; k' <= 256 candidates (slots 0..3) + K <= 128 list entries (slots 4, 5) per lane
template <typename IN>
__global__ void __launch_bounds__(GR_NT)
gr_merge_kernel(const IN *__restrict__ Wl, int64_t C_loc, const IN *__restrict__ Wv, int64_t C_vis, int D, int K, int cap,
                const uint64_t *__restrict__ cand, const int32_t *__restrict__ cnt, const uint32_t *__restrict__ thr,
                const float *__restrict__ norms, const float *__restrict__ maxnorm, float gamma, int64_t local_offset,
                int64_t visit_offset, int32_t *__restrict__ graph, double *__restrict__ sims, int32_t *fb_count,
                int32_t *__restrict__ fb_rows) {
    const int64_t i = (int64_t)blockIdx.x * (GR_NT / 64) + (threadIdx.x >> 6);
    if (i >= C_loc) return;
    const int lane = threadIdx.x & 63;
    const int n = cnt[i];
    double s[6];
    int32_t id[6];
#pragma unroll
    for (int t = 4; t < 6; ++t) { // the list so far
        const int e = (t - 4) * 64 + lane;
        s[t] = -INFINITY;
        id[t] = GR_NO_ID;
        if (e < K) {
            const int32_t g = graph[i * K + e];
            if (g >= 0) {
                id[t] = g;
                s[t] = sims[i * K + e];
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) { // the recalled candidates
        const int q = t * 64 + lane;
        s[t] = -INFINITY;
        id[t] = GR_NO_ID;
        if (q < n) {
            const uint32_t j = 0xFFFFFFFFu - (uint32_t)cand[i * cap + q];
            if (j < (uint64_t)C_vis) { // always true for keys written by the recall pass
                id[t] = (int32_t)(visit_offset + j);
                s[t] = gr_canon(Wl + i * D, Wv + (int64_t)j * D, D);
            }
        }
    }
    // a visiting row that is in the list already (a shard seen twice) is not a new candidate
    const int list_slots = (K + 63) >> 6;
    for (int t2 = 0; t2 < list_slots; ++t2) {
        const int32_t mine = t2 == 0 ? id[4] : id[5];
        for (int src = 0; src < 64; ++src) {
            const int32_t oid = __shfl(mine, src, 64);
            if (oid == GR_NO_ID) continue;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (id[t] == oid) {
                    id[t] = GR_NO_ID;
                    s[t] = -INFINITY;
                }
        }
    }
    int rank[6] = {0, 0, 0, 0, 0, 0};
    int n_valid = 0;
    const int cand_slots = (n + 63) >> 6;
#pragma unroll
    for (int t2 = 0; t2 < 6; ++t2) {
        if (t2 < 4 ? t2 >= cand_slots : t2 - 4 >= list_slots) continue; // uniform over the wavefront
        n_valid += __popcll(__ballot(id[t2] != GR_NO_ID));
        for (int src = 0; src < 64; ++src) {
            const double os = __shfl(s[t2], src, 64);
            const int32_t oid = __shfl(id[t2], src, 64);
            if (oid == GR_NO_ID) continue;
#pragma unroll
            for (int t = 0; t < 6; ++t) rank[t] += gr_ranks_before(os, oid, s[t], id[t]) ? 1 : 0;
        }
    }
    bool certified = true;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        if (id[t] != GR_NO_ID && rank[t] < K) {
            graph[i * K + rank[t]] = id[t];
            sims[i * K + rank[t]] = s[t];
            if (rank[t] == K - 1) {
                // certificate: no visiting row that the recall pass dropped can reach the K-th exact similarity
                const uint32_t th = thr[i];
                if (th != 0u) {
                    const double eps = (double)gamma * (double)norms[i] * (double)*maxnorm;
                    certified = s[t] > (double)gr_unorder(th) + eps;
                }
            }
        }
    }
    for (int e = n_valid + lane; e < K; e += 64) { // fewer than K known so far: empty slots
        graph[i * K + e] = -1;
        sims[i * K + e] = -INFINITY;
    }
    if (n_valid < K && thr[i] != 0u) certified = false; // cannot happen (something was dropped, so k' >= K were kept)
    if (__ballot(!certified) != 0ull && lane == 0) fb_rows[atomicAdd(fb_count, 1)] = (int32_t)i;
}

__global__ void __launch_bounds__(GR_NT)
gr_hop_threshold_kernel(int64_t C_loc, GrHop hop, const float *__restrict__ maxnorm, uint32_t *__restrict__ thr) {
    const int64_t i = (int64_t)blockIdx.x * GR_NT + threadIdx.x;
    if (i < C_loc) thr[i] = gr_hop_threshold(hop, i, *maxnorm);
}

// rows on the list: every visiting row in canonical fp64 arithmetic, merged with the row's list
template <typename IN>
__global__ void __launch_bounds__(GR_NT)
gr_exhaustive_merge_kernel(const IN *__restrict__ Wl, int64_t C_loc, const IN *__restrict__ Wv, int64_t C_vis, int D, int K,
                           int64_t local_offset, int64_t visit_offset, const int32_t *__restrict__ fb_count,
                           const int32_t *__restrict__ fb_rows, double *__restrict__ scratch, int32_t *__restrict__ graph,
                           double *__restrict__ sims) {
    __shared__ double red_s[GR_NT];
    __shared__ int32_t red_j[GR_NT];
    __shared__ __attribute__((aligned(16))) IN row_i[GR_MAX_D];
    __shared__ double l_s[KS_MAX_GRAPH_K], o_s[KS_MAX_GRAPH_K];
    __shared__ int32_t l_id[KS_MAX_GRAPH_K], o_id[KS_MAX_GRAPH_K];
    int n_fb = *fb_count;
    if (n_fb > C_loc) n_fb = (int)C_loc;
    double *my = scratch + (int64_t)blockIdx.x * C_vis;
    for (int e = blockIdx.x; e < n_fb; e += gridDim.x) {
        const int64_t i = fb_rows[e];
        for (int d = threadIdx.x; d < D; d += GR_NT) row_i[d] = Wl[i * D + d];
        for (int k = threadIdx.x; k < K; k += GR_NT) {
            l_id[k] = graph[i * K + k];
            l_s[k] = sims[i * K + k];
        }
        __syncthreads();
        for (int64_t j = threadIdx.x; j < C_vis; j += GR_NT) my[j] = gr_canon(row_i, Wv + j * D, D);
        __syncthreads();
        // the row itself and visiting rows that are in the list already are no candidates (-inf marks them: the
        // similarity of real rows is finite)
        if (threadIdx.x == 0) {
            const int64_t js = local_offset + i - visit_offset;
            if (js >= 0 && js < C_vis) my[js] = -INFINITY;
        }
        for (int k = threadIdx.x; k < K; k += GR_NT) {
            const int64_t jl = (int64_t)l_id[k] - visit_offset;
            if (l_id[k] >= 0 && jl >= 0 && jl < C_vis) my[jl] = -INFINITY;
        }
        __syncthreads();
        double prev_s = INFINITY;
        int32_t prev_j = -1;
        for (int r = 0; r < K; ++r) {
            double best_s = -INFINITY;
            int32_t best_j = GR_NO_ID;
            for (int64_t j = threadIdx.x; j < C_vis; j += GR_NT) {
                const double sj = my[j];
                if (sj == -INFINITY) continue;
                const int32_t gj = (int32_t)(visit_offset + j);
                if (gr_ranks_before(prev_s, prev_j, sj, gj) && gr_ranks_before(sj, gj, best_s, best_j)) {
                    best_s = sj;
                    best_j = gj;
                }
            }
            for (int k = threadIdx.x; k < K; k += GR_NT) {
                if (l_id[k] < 0) continue;
                if (gr_ranks_before(prev_s, prev_j, l_s[k], l_id[k]) && gr_ranks_before(l_s[k], l_id[k], best_s, best_j)) {
                    best_s = l_s[k];
                    best_j = l_id[k];
                }
            }
            red_s[threadIdx.x] = best_s;
            red_j[threadIdx.x] = best_j;
            __syncthreads();
            for (int o = GR_NT / 2; o > 0; o >>= 1) {
                if (threadIdx.x < o) {
                    if (gr_ranks_before(red_s[threadIdx.x + o], red_j[threadIdx.x + o], red_s[threadIdx.x], red_j[threadIdx.x])) {
                        red_s[threadIdx.x] = red_s[threadIdx.x + o];
                        red_j[threadIdx.x] = red_j[threadIdx.x + o];
                    }
                }
                __syncthreads();
            }
            prev_s = red_s[0];
            prev_j = red_j[0];
            if (threadIdx.x == 0) {
                o_id[r] = prev_j == GR_NO_ID ? -1 : prev_j;
                o_s[r] = prev_j == GR_NO_ID ? -INFINITY : prev_s;
            }
            __syncthreads();
            if (prev_j == GR_NO_ID) { // nothing left: the remaining slots are empty
                for (int k = r + 1 + threadIdx.x; k < K; k += GR_NT) { o_id[k] = -1; o_s[k] = -INFINITY; }
                break;
            }
        }
        __syncthreads();
        for (int k = threadIdx.x; k < K; k += GR_NT) {
            graph[i * K + k] = o_id[k];
            sims[i * K + k] = o_s[k];
        }
        __syncthreads();
    }
}

struct GrUpWs {
    uint16_t *Wlb, *Wvb;
    float *norms_l, *blockmax_l, *blockmax_v, *maxnorm_v;
    uint64_t *cand;
    int32_t *fb_count;
    int32_t *fb_rows;
    double *scratch;
    int32_t *cnt;  // running thresholds
    uint32_t *thr;
    uint16_t *Ws;  // fixed thresholds
    float *tops, *thf;
    uint32_t *tbits;
    int32_t *cnt_res;
};
static GrUpWs gr_up_carve(void *ws, int64_t C_loc, int64_t C_vis, int D, int K, int dtype, size_t *total) {
    KsArena ar(ws);
    GrParams p = gr_params(K, D);
    GrUpWs w = GrUpWs();
    w.Wlb = dtype == KS_DTYPE_FP32 ? ar.take<uint16_t>((size_t)C_loc * D) : nullptr;
    w.Wvb = dtype == KS_DTYPE_FP32 ? ar.take<uint16_t>((size_t)C_vis * D) : nullptr;
    w.norms_l = ar.take<float>((size_t)C_loc);
    w.blockmax_l = ar.take<float>(GR_PREP_BLOCKS);
    w.blockmax_v = ar.take<float>(GR_PREP_BLOCKS);
    w.maxnorm_v = ar.take<float>(1);
    w.fb_count = ar.take<int32_t>(1);
    w.fb_rows = ar.take<int32_t>((size_t)C_loc);
    w.scratch = ar.take<double>((size_t)GR_FB_BLOCKS * C_vis);
    if (gr_use_fixed(C_loc, C_vis, D, K)) {
        const GrFixPlan f = gr_fix_plan(C_loc, C_vis, D, K, dtype, false, true);
        w.cand = ar.take<uint64_t>((size_t)C_loc * f.room);
        KsArena over(w.scratch);
        w.Ws = over.take<uint16_t>((size_t)(C_vis / f.every) * D);
        w.tops = f.smp.parts > 1 ? over.take<float>((size_t)f.smp.parts * GR_RANK * C_loc) : nullptr;
        w.thf = ar.take<float>((size_t)C_loc);
        w.tbits = ar.take<uint32_t>((size_t)C_loc);
        w.cnt_res = ar.take<int32_t>((size_t)C_loc * 2 * f.room_parts);
    } else {
        w.cand = ar.take<uint64_t>((size_t)C_loc * p.cap);
        w.cnt = ar.take<int32_t>((size_t)C_loc);
        w.thr = ar.take<uint32_t>((size_t)C_loc);
    }
    if (total) *total = ar.off;
    return w;
}
static int gr_up_check(int64_t C_loc, int64_t C_vis, int D, int K, int dtype, int64_t lo, int64_t vo) {
    if (dtype != KS_DTYPE_BF16 && dtype != KS_DTYPE_FP32) return KS_INVALID_ARG;
    if (C_loc < 1 || C_vis < 1 || D < 32 || D % 32 != 0 || K < 1 || lo < 0 || vo < 0) return KS_INVALID_ARG;
    if (lo + C_loc >= (int64_t)1 << 31 || vo + C_vis >= (int64_t)1 << 31) return KS_INVALID_ARG;
    if (K > KS_MAX_GRAPH_K || D > GR_MAX_D) return KS_UNSUPPORTED;
    return KS_OK;
}

extern "C" size_t knn_graph_update_workspace(int64_t C_loc, int64_t C_vis, int D, int K, int dtype) {
    if (gr_up_check(C_loc, C_vis, D, K, dtype, 0, 0) != KS_OK) return 0;
    size_t total = 0;
    gr_up_carve(nullptr, C_loc, C_vis, D, K, dtype, &total);
    return total;
}

template <typename IN>
static void gr_up_exact(const IN *Wl, int64_t C_loc, const IN *Wv, int64_t C_vis, int D, int K, const GrParams &p, const GrFixPlan *f,
                        const GrUpWs &w, float gamma, int64_t lo, int64_t vo, int32_t *graph, double *sims, hipStream_t st) {
    const dim3 grid((unsigned)ks_ceil_div(C_loc, GR_NT / 64));
#define GR_HOP_RANK_LAUNCH(KP, SHORT, LANES)                                                                                   \
    hipLaunchKernelGGL((gr_rank_kernel<IN, KP, true, SHORT, LANES>), grid, dim3(GR_NT), 0, st, Wl, C_loc, Wv, C_vis, D, K, f->seg,      \
                       w.cand, w.cnt_res, (const int32_t *)nullptr, w.tbits, w.norms_l, w.maxnorm_v, gamma, vo, graph, (void *)sims, \
                       w.fb_count, w.fb_rows)
    if (f && K <= 24 && C_loc > GR_RANK_AT_ONCE) GR_HOP_RANK_LAUNCH(1, true, true);
    else if (f && (K <= 29 || (K <= 32 && D <= 128))) GR_HOP_RANK_LAUNCH(1, false, true);
    else if (f && K <= 32) GR_HOP_RANK_LAUNCH(1, false, sizeof(IN) == 2);
    else if (f && sizeof(IN) == 2 && C_loc > GR_RANK_AT_ONCE) GR_HOP_RANK_LAUNCH(2, true, false);
    else if (f) GR_HOP_RANK_LAUNCH(2, false, false);
    else
        hipLaunchKernelGGL(gr_merge_kernel<IN>, grid, dim3(GR_NT), 0, st, Wl, C_loc, Wv, C_vis, D, K, p.cap, w.cand, w.cnt, w.thr,
                           w.norms_l, w.maxnorm_v, gamma, lo, vo, graph, sims, w.fb_count, w.fb_rows);
#undef GR_HOP_RANK_LAUNCH
    hipLaunchKernelGGL(gr_exhaustive_merge_kernel<IN>, dim3(GR_FB_BLOCKS), dim3(GR_NT), 0, st, Wl, C_loc, Wv, C_vis, D, K, lo, vo,
                       w.fb_count, w.fb_rows, w.scratch, graph, sims);
}

extern "C" int knn_graph_recall_plan(int64_t C_loc, int64_t C_vis, int D, int K, int dtype, int32_t *out) {
    if (!out) return KS_INVALID_ARG;
    const bool hop = C_vis != 0;
    const int rc = hop ? gr_up_check(C_loc, C_vis, D, K, dtype, 0, 0) : gr_check(C_loc, D, K, dtype);
    if (rc != KS_OK) return rc;
    const int64_t Cs = hop ? C_vis : C_loc;
    const bool sym = !hop && gr_use_sym(C_loc, D, K);
    for (int q = 0; q < 5; ++q) out[q] = 0;
    if (!gr_use_fixed(C_loc, Cs, D, K)) return KS_OK;
    out[0] = sym ? 2 : 1;
    if (sym) return KS_OK;
    const GrFixPlan f = gr_fix_plan(C_loc, Cs, D, K, dtype, false, hop);
    out[1] = f.seg.parts;
    out[2] = f.part_rows;
    out[3] = f.turns ? gr_chunk(D) : 96;
    out[4] = f.turns ? 1 : 0;
    return KS_OK;
}

extern "C" int knn_graph_update(const void *W_local, const void *W_visit, int dtype, int64_t C_loc, int64_t C_vis, int D, int K,
                                int64_t local_offset, int64_t visit_offset, int32_t *graph, double *sims, void *ws,
                                size_t ws_bytes, int32_t *dev_status, void *stream) {
    (void)dev_status;
    if (!W_local || !W_visit || !graph || !sims || !ws) return KS_INVALID_ARG;
    int rc = gr_up_check(C_loc, C_vis, D, K, dtype, local_offset, visit_offset);
    if (rc != KS_OK) return rc;
    size_t need = 0;
    GrUpWs w = gr_up_carve(ws, C_loc, C_vis, D, K, dtype, &need);
    if (ws_bytes < need) return KS_WORKSPACE_TOO_SMALL;
    const GrParams p = gr_params(K, D, dtype);
    hipStream_t st = (hipStream_t)stream;
    const bool fixed = gr_use_fixed(C_loc, C_vis, D, K);
    const GrFixPlan f = gr_fix_plan(C_loc, C_vis, D, K, dtype, false, true);
    GrClear clr = GrClear();
    clr.fb_count = w.fb_count;
    const GrPrepJob jl = gr_prep_job(W_local, C_loc, D, dtype, w.Wlb, w.norms_l, w.blockmax_l, nullptr, 0);
    const GrPrepJob jv = gr_prep_job(W_visit, C_vis, D, dtype, w.Wvb, nullptr, w.blockmax_v, fixed ? w.Ws : nullptr, f.every);
    gr_launch_prepare(jl, jv, D, dtype, clr, st);
    const uint16_t *Rl = dtype == KS_DTYPE_FP32 ? w.Wlb : (const uint16_t *)W_local;
    const uint16_t *Sv = dtype == KS_DTYPE_FP32 ? w.Wvb : (const uint16_t *)W_visit;
    const GrPair pr{Rl, C_loc, Sv, C_vis, local_offset - visit_offset};
    const float gamma = gr_gamma(D, dtype);
    const GrHop hop{graph, sims, w.norms_l, K, gamma};
    if (fixed) {
        GrSample smp = f.smp;
        smp.tops = w.tops;
        gr_launch_threshold(Rl, C_loc, w.Ws, jv.n_sample, D, smp, w.blockmax_v, jv.blocks, w.maxnorm_v, hop, w.thf, w.tbits, st);
        gr_launch_recall_fix(pr, D, f, smp, hop, w.maxnorm_v, w.thf, w.tbits, w.cand, w.cnt_res, st);
    } else {
        hipLaunchKernelGGL(gr_maxnorm_kernel, dim3(1), dim3(64), 0, st, w.blockmax_v, jv.blocks, w.maxnorm_v);
        hipLaunchKernelGGL(gr_hop_threshold_kernel, dim3((unsigned)ks_ceil_div(C_loc, GR_NT)), dim3(GR_NT), 0, st, C_loc, hop,
                           w.maxnorm_v, w.thr);
        gr_launch_recall(pr, D, p, w.cand, w.cnt, w.thr, st, w.thr);
    }
    const GrFixPlan *fp = fixed ? &f : nullptr;
    if (dtype == KS_DTYPE_FP32)
        gr_up_exact<float>((const float *)W_local, C_loc, (const float *)W_visit, C_vis, D, K, p, fp, w, gamma, local_offset,
                           visit_offset, graph, sims, st);
    else
        gr_up_exact<uint16_t>((const uint16_t *)W_local, C_loc, (const uint16_t *)W_visit, C_vis, D, K, p, fp, w, gamma,
                              local_offset, visit_offset, graph, sims, st);
    KS_LAUNCH_CHECK();
    return KS_OK;
}
