// KNN-softmax forward + backward on the active classes (paper Section 3.2; Section 3.1 steps 3-5).
//
// Pipeline on one stream (A = number of active classes, known only on the device):
//   select            -> active_idx, n_active, target_pos                         (ks_select.hip)
//   logits GEMM       Z[B, A]  = scale * X . W[active]^T     rows of W fetched through the index list
//   row statistics    lse_i, loss_i                           one workgroup per sample
//   loss mean         fixed-order tree sum
//   logit gradient    dZ[B, A] = g (exp(Z - lse) - onehot)    bf16
//   dX GEMM           split over the active dimension, partial tiles summed in a fixed order
//   dW GEMM           dW_active[A, D] = scale * dZ^T . X
// Launch sizes are taken from the cap M; workgroups beyond the active count exit at once.
#include "ks_gemm.h"
#include "ks_gemm_async.h"
#include "ks_gemm_soe.h"
#include "ks_select.h"

typedef KsTile<128, 128, 64, 2, 2> TileG;      // generic path (any D % 32 == 0)
typedef KsATile<256, 256, 2, 4, 2> TileSm;     // fast path (D % 64 == 0): tile = 256 classes x 256 samples
typedef KsATile<128, 128, 2, 2, 2, KS_K8> TileDx;
typedef KsATile<256, 256, 2, 4, 2, KS_K8> TileDxWide; // see sm_dx_wide
// gather indices of one workgroup's share of the active dimension, staged in LDS
template <class T> struct DxIdx { static constexpr int CAP = T::BM == 256 ? 8192 : 4096; };
// dW tiles (active rows x columns of D): chosen inside the kernel from the number of active rows, which only the device
// knows (see dw_tile_kind)
typedef KsATile<256, 256, 2, 4, 2, KS_M8> TileDw;
typedef KsATile<192, 256, 2, 4, 2, KS_M8> TileDw192;
typedef KsATile<128, 256, 2, 4, 2, KS_M8> TileDw128;
typedef KsATile<128, 128, 2, 4, 2, KS_M8> TileDw128n; // (n: 128 columns)
typedef KsATile<64, 128, 2, 4, 2, KS_M8> TileDw64n;
#define KS_BP_ALIGN 256
#define SM_LIDX_CAP 1536 // gather-list entries a sweep keeps in LDS (longer slabs read the list from memory)
#define SM_SOE_GRID 256 /* workgroups of the stationary-operand softmax passes (one per compute unit) */

#define SM_NT 256
#define KS_MP_ALIGN 256

static inline int64_t sm_mp(int64_t M) { return (int64_t)ks_align_up((size_t)M, KS_MP_ALIGN); }

__device__ __forceinline__ int sm_clamp_n(const int32_t *n_active, int M) {
    int n = *n_active;
    return n < 0 ? 0 : (n > M ? M : n);
}

// ------------------------------------------------------------------------------------------------
// Z = scale * X . W[active]^T      (M index = sample i, N index = active position a, K index = d)
// ------------------------------------------------------------------------------------------------
template <class T>
__global__ void __launch_bounds__(T::NT)
logits_kernel(const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, const int32_t *__restrict__ active_idx,
              const int32_t *__restrict__ n_active_p, int B, int D, int M, float scale, float *__restrict__ Z,
              int64_t ldz) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::LDS_ELEMS];
    const int n_active = sm_clamp_n(n_active_p, M);
    const int tiles_m = (B + T::BM - 1) / T::BM;
    const int n_tiles = tiles_m * ((n_active + T::BN - 1) / T::BN);
    if ((int)blockIdx.x >= n_tiles) return;
    const int t = ks_xcd_remap(blockIdx.x, n_tiles);
    const int tm = t % tiles_m, tn = t / tiles_m;

    KsRowLoader<T::BM, T::BK, T::NT> al;
    KsRowLoader<T::BN, T::BK, T::NT> bl;
    al.init(X, D, nullptr, tm * T::BM, B, D);
    bl.init(W, D, active_idx, tn * T::BN, n_active, D);
    f32x16_t acc[T::FM][T::FN];
    ks_tile_clear<T>(acc);
    ks_gemm_mainloop<T>(al, bl, 0, (D + T::BK - 1) / T::BK, lds, acc);
    ks_tile_foreach<T>(acc, [&](int m, int n, float v) {
        int i = tm * T::BM + m, a = tn * T::BN + n;
        if (i < B && a < n_active) Z[(int64_t)i * ldz + a] = scale * v;
    });
}

// ------------------------------------------------------------------------------------------------
// per-sample log-sum-exp and loss; one workgroup per sample
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(SM_NT)
row_stats_kernel(const float *__restrict__ Z, int64_t ldz, const int32_t *__restrict__ n_active_p, int M,
                 const int32_t *__restrict__ target_pos, float *__restrict__ lse_out, float *__restrict__ loss_i) {
    __shared__ float sm[SM_NT / 64], sl[SM_NT / 64];
    const int i = blockIdx.x;
    const int n = sm_clamp_n(n_active_p, M);
    const float *z = Z + (int64_t)i * ldz;
    float m = -INFINITY, l = 0.f;
    const int n4 = n & ~3;
    for (int a = threadIdx.x * 4; a < n4; a += SM_NT * 4) {
        float4 v = *(const float4 *)(z + a);
        float mx = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
        if (mx > m) { l *= __expf(m - mx); m = mx; }
        l += __expf(v.x - m) + __expf(v.y - m) + __expf(v.z - m) + __expf(v.w - m);
    }
    if (threadIdx.x < n - n4) {
        float v = z[n4 + threadIdx.x];
        if (v > m) { l *= __expf(m - v); m = v; }
        l += __expf(v - m);
    }
    // combine (m, l) pairs: wave, then block, in a fixed order
    float wm = ks_wave_max(m);
    float wl = ks_wave_sum(m == -INFINITY ? 0.f : l * __expf(m - wm));
    if ((threadIdx.x & 63) == 0) { sm[threadIdx.x >> 6] = wm; sl[threadIdx.x >> 6] = wl; }
    __syncthreads();
    if (threadIdx.x == 0) {
        float bm = sm[0];
        for (int w = 1; w < SM_NT / 64; ++w) bm = fmaxf(bm, sm[w]);
        float bl = 0.f;
        for (int w = 0; w < SM_NT / 64; ++w) bl += (sm[w] == -INFINITY) ? 0.f : sl[w] * __expf(sm[w] - bm);
        float lse = bm + __logf(bl);
        int tp = target_pos[i];
        float zt = (tp >= 0 && tp < n) ? z[tp] : 0.f;
        lse_out[i] = lse;
        loss_i[i] = lse - zt;
    }
}

// (The mean of the per-sample losses is formed later in the stream, by one block of dx_reduce_kernel: folding
// it into the kernel above would need a device-scope fence per workgroup, which costs far more on this chip,
// whose eight L2 caches are only coherent through memory, and a launch of its own costs about 5 us.)

// ------------------------------------------------------------------------------------------------
// dZ = g (exp(Z - lse) - onehot) as bf16; columns in [n_active, round_up(n_active, 256)) are zeroed
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(SM_NT)
dz_kernel(const float *__restrict__ Z, int64_t ldz, const int32_t *__restrict__ n_active_p, int B, int M,
          const int32_t *__restrict__ target_pos, const float *__restrict__ lse, float g, uint16_t *__restrict__ dZ) {
    const int n = sm_clamp_n(n_active_p, M);
    const int n_pad = (n + KS_MP_ALIGN - 1) / KS_MP_ALIGN * KS_MP_ALIGN; // <= ldz
    const int a0 = (blockIdx.x * SM_NT + threadIdx.x) * 8;
    if (a0 >= n_pad) return;
    for (int i = blockIdx.y; i < B; i += gridDim.y) { // (the y dimension of a grid ends at 65,535)
        const float ls = lse[i];
        const int tp = target_pos[i];
        const float *z = Z + (int64_t)i * ldz + a0;
        float v[8];
        if (a0 + 8 <= n) {
            float4 p = *(const float4 *)z, q = *(const float4 *)(z + 4);
            v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = p.w; v[4] = q.x; v[5] = q.y; v[6] = q.z; v[7] = q.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = (a0 + e < n) ? z[e] : 0.f;
        }
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            float d0 = (a0 + e < n) ? g * (__expf(v[e] - ls) - (a0 + e == tp ? 1.f : 0.f)) : 0.f;
            float d1 = (a0 + e + 1 < n) ? g * (__expf(v[e + 1] - ls) - (a0 + e + 1 == tp ? 1.f : 0.f)) : 0.f;
            o[e / 2] = ks_pack_bf2(d0, d1);
        }
        *(uint4 *)(dZ + (int64_t)i * ldz + a0) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

// ------------------------------------------------------------------------------------------------
// dX partials: P[s][i][d] = sum over the s-th share of a of dZ[i][a] * W[active[a]][d]
// ------------------------------------------------------------------------------------------------
template <class T>
__global__ void __launch_bounds__(T::NT)
dx_partial_kernel(const uint16_t *__restrict__ dZ, int64_t ldz, const uint16_t *__restrict__ W,
                  const int32_t *__restrict__ active_idx, const int32_t *__restrict__ n_active_p, int B, int D, int M,
                  float *__restrict__ part) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::LDS_ELEMS];
    const int n_active = sm_clamp_n(n_active_p, M);
    const int tiles_m = (B + T::BM - 1) / T::BM;
    const int tm = blockIdx.x % tiles_m, tn = blockIdx.x / tiles_m;
    const int s = blockIdx.y, S = gridDim.y;
    const int nk = (n_active + T::BK - 1) / T::BK;
    const int per = (nk + S - 1) / S;
    const int kt0 = s * per, kt1 = (kt0 + per < nk) ? kt0 + per : nk;

    KsRowLoader<T::BM, T::BK, T::NT> al;
    KsColLoader<T::BN, T::BK, T::NT> bl;
    al.init(dZ, ldz, nullptr, tm * T::BM, B, (n_active + 7) & ~7);
    bl.init(W, D, active_idx, tn * T::BN, D, n_active);
    f32x16_t acc[T::FM][T::FN];
    ks_tile_clear<T>(acc);
    ks_gemm_mainloop<T>(al, bl, kt0, kt1, lds, acc);
    float *out = part + (int64_t)s * B * D;
    ks_tile_foreach<T>(acc, [&](int m, int n, float v) {
        int i = tm * T::BM + m, d = tn * T::BN + n;
        if (i < B && d < D) out[(int64_t)i * D + d] = v;
    });
}

__global__ void __launch_bounds__(SM_NT)
dx_reduce_kernel(const float *__restrict__ part, int S, int64_t BD, float scale, const float *__restrict__ row_factor,
                 int D, float *__restrict__ dX, const float *__restrict__ loss_i, int B, float *loss_mean) {
    // the last block also folds the per-sample losses (complete since an earlier launch) into the batch
    // mean: thread t takes samples t, t + SM_NT, ..., then a tree -- a fixed order, and no launch of its own
    if (loss_mean && blockIdx.x == gridDim.x - 1) {
        __shared__ float sh[SM_NT];
        float s = 0.f;
        for (int i = threadIdx.x; i < B; i += SM_NT) s += loss_i[i];
        sh[threadIdx.x] = s;
        __syncthreads();
        for (int o = SM_NT / 2; o > 0; o >>= 1) {
            if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss_mean = sh[0] / (float)B;
    }
    int64_t e = ((int64_t)blockIdx.x * SM_NT + threadIdx.x) * 4;
    if (e >= BD) return; // BD % 4 == 0, D % 4 == 0
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < S; ++s) {
        float4 v = *(const float4 *)(part + (int64_t)s * BD + e);
        acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    if (row_factor) scale *= row_factor[e / D]; // per-sample factor (the one-sweep softmax leaves 1 / sum there)
    *(float4 *)(dX + e) = make_float4(scale * acc.x, scale * acc.y, scale * acc.z, scale * acc.w);
}

// ------------------------------------------------------------------------------------------------
// dW_active[a][d] = scale * sum_i dZ[i][a] * X[i][d]     (both operands k-major: k = i)
// ------------------------------------------------------------------------------------------------
template <class T>
__global__ void __launch_bounds__(T::NT)
dw_kernel(const uint16_t *__restrict__ dZ, int64_t ldz, const uint16_t *__restrict__ X,
          const int32_t *__restrict__ n_active_p, int B, int D, int M, float scale, float *__restrict__ dW) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::LDS_ELEMS];
    const int n_active = sm_clamp_n(n_active_p, M);
    const int tiles_n = (D + T::BN - 1) / T::BN;
    const int n_tiles = tiles_n * ((n_active + T::BM - 1) / T::BM);
    if ((int)blockIdx.x >= n_tiles) return;
    const int t = ks_xcd_remap(blockIdx.x, n_tiles);
    const int tn = t % tiles_n, tm = t / tiles_n;

    KsColLoader<T::BM, T::BK, T::NT> al;
    KsColLoader<T::BN, T::BK, T::NT> bl;
    al.init(dZ, ldz, nullptr, tm * T::BM, (int)ldz, B);
    bl.init(X, D, nullptr, tn * T::BN, D, B);
    f32x16_t acc[T::FM][T::FN];
    ks_tile_clear<T>(acc);
    ks_gemm_mainloop<T>(al, bl, 0, (B + T::BK - 1) / T::BK, lds, acc);
    ks_tile_foreach<T>(acc, [&](int m, int n, float v) {
        int a = tm * T::BM + m, d = tn * T::BN + n;
        if (a < n_active && d < D) dW[(int64_t)a * D + d] = scale * v;
    });
}

// ================================================================================================
// Fast path (D <= 512, or D % 64 == 0).  The contractions run on the asynchronous and the stationary-operand engine and the
// logits are recomputed instead of stored (see below).  The logit gradient is stored once, in blocks of eight classes:
//     dZ8[(a / 8) * Bp + i][a % 8]        (Bp: samples rounded up to whole tiles)
// In the accumulators of the sweeps a lane holds four consecutive classes of one sample, so a block's 16 bytes come together
// by exchanging halves between two lanes (v_permlane32_swap) and leave as full 512-byte rows straight from registers: no
// transposition through LDS.  For the dX contraction (over classes) such a block is a ready MFMA fragment; the dW contraction
// (over samples) reads the same array through the transposing LDS read.  Weight rows (gathered through the index list) and
// X enter as k-major operands where k is their row index, so no transposed copies of them are made.
// ================================================================================================

// element (class position a, sample i) of dZ8
__device__ __forceinline__ int64_t sm_dz_at(int a, int i, int Bp) { return (((int64_t)(a >> 3) * Bp) + i) * 8 + (a & 7); }

// Stores the values of one 32 x 32 accumulator block as bf16: pk[g] = the lane's classes 8 g + 4 (lane / 32) .. + 3 of its
// sample, packed in pairs.  p: the lane's sample in the block of eight classes (lane / 32) of the accumulator block.
// After the exchange a lane holds all eight classes of its sample for block 0 or 2 (lanes 0..31) or 1 or 3 (lanes 32..63).
__device__ __forceinline__ void sm_store_block(uint32_t (&pk)[4][2], uint16_t *p, int Bp) {
#pragma unroll
    for (int g = 0; g < 4; g += 2) {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const auto x = __builtin_amdgcn_permlane32_swap(pk[g][w], pk[g + 1][w], false, false);
            pk[g][w] = x[0];
            pk[g + 1][w] = x[1];
        }
        *(uint4 *)(p + (int64_t)g * Bp * 8) = make_uint4(pk[g][0], pk[g][1], pk[g + 1][0], pk[g + 1][1]);
    }
}

// Only small problems store their logits on the fast path (sm_kept_bytes).  Two passes over the same tile product
//     Zt[a][i] = scale * <W[active[a]], X[i]>            (classes = MFMA rows, samples = MFMA columns)
// First pass: per-sample running max / sum of exponentials of each class tile, and the target logit.
// Second pass (after the per-sample log-sum-exp is known): the same product again, turned into the logit
// gradient in registers and stored transposed, dZ8[a][i].  In this orientation a lane owns one sample
// column of the accumulator tile, so the per-sample reductions are lane-local.

// accumulator element (fm, r) of a lane: class row inside the wave's part of the tile
__device__ __forceinline__ int sm_tile_row(int fm, int r, int lane) { return fm * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

template <class T>
__device__ __forceinline__ void sm_logits_tile(const uint16_t *X, const uint16_t *W, const int32_t *active_idx, int n_active,
                                               int B, int D, int tc, int ts, uint16_t *lds, f32x16_t (&acc)[T::FM][T::FN]) {
    KsARows<T::BM, T::NW> ar;
    KsARows<T::BN, T::NW> br;
    ar.init(W, D, active_idx, tc * T::BM, n_active);
    br.init(X, D, nullptr, ts * T::BN, B);
    ks_a_clear<T>(acc);
    ks_a_mainloop<T>(ar, br, 0, D / 64, lds, acc);
}

template <class T>
__global__ void __launch_bounds__(T::NT)
sm_stats_kernel(const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, const int32_t *__restrict__ active_idx,
                const int32_t *__restrict__ n_active_p, const int32_t *__restrict__ target_pos, int B, int Bp, int D, int M,
                float scale, float *__restrict__ pm, float *__restrict__ pl, float *__restrict__ zt) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::LDS_ELEMS];
    const int n_active = sm_clamp_n(n_active_p, M);
    const int tiles_s = (B + T::BN - 1) / T::BN;
    const int n_tiles = tiles_s * ((n_active + T::BM - 1) / T::BM);
    if ((int)blockIdx.x >= n_tiles) return;
    const int t = ks_xcd_remap(blockIdx.x, n_tiles);
    const int ts = t % tiles_s, tc = t / tiles_s;
    f32x16_t acc[T::FM][T::FN];
    sm_logits_tile<T>(X, W, active_idx, n_active, B, D, tc, ts, lds, acc); // ends with a barrier: LDS is free

    // per (wave row, sample) partial statistics go through LDS: [WAVES_M][BN] pairs
    float *s_m = (float *)lds, *s_l = s_m + T::WAVES_M * T::BN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / T::WAVES_N, wn = wave % T::WAVES_N;
    const int c0 = tc * T::BM + wm * T::WM;
#pragma unroll
    for (int fn = 0; fn < T::FN; ++fn) {
        const int col = wn * T::WN + fn * 32 + (lane & 31);
        const int i = ts * T::BN + col;
        const int tp = (i < B) ? target_pos[i] : -1;
        float m = -INFINITY;
#pragma unroll
        for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int c = c0 + sm_tile_row(fm, r, lane);
                const float z = scale * acc[fm][fn][r];
                if (c < n_active) m = fmaxf(m, z);
                if (c == tp) zt[i] = z;
            }
        float l = 0.f;
#pragma unroll
        for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int c = c0 + sm_tile_row(fm, r, lane);
                if (c < n_active) l += __expf(scale * acc[fm][fn][r] - m);
            }
        // the two half-waves hold disjoint class rows of the same 32 samples
        const float mo = __shfl_xor(m, 32, 64), lo = __shfl_xor(l, 32, 64);
        const float mm = fmaxf(m, mo);
        const float ll = (m == -INFINITY ? 0.f : l * __expf(m - mm)) + (mo == -INFINITY ? 0.f : lo * __expf(mo - mm));
        if (lane < 32) {
            s_m[wm * T::BN + col] = mm;
            s_l[wm * T::BN + col] = ll;
        }
    }
    __syncthreads();
    for (int col = threadIdx.x; col < T::BN; col += T::NT) {
        const int i = ts * T::BN + col;
        if (i >= B) continue;
        float mm = s_m[col], ll = s_l[col];
#pragma unroll
        for (int w = 1; w < T::WAVES_M; ++w) { // fixed order
            const float m2 = s_m[w * T::BN + col], l2 = s_l[w * T::BN + col];
            const float mx = fmaxf(mm, m2);
            ll = (mm == -INFINITY ? 0.f : ll * __expf(mm - mx)) + (m2 == -INFINITY ? 0.f : l2 * __expf(m2 - mx));
            mm = mx;
        }
        pm[(int64_t)tc * Bp + i] = mm;
        pl[(int64_t)tc * Bp + i] = ll;
    }
}

// one wavefront per sample: merge the per-tile (max, sum) pairs in tile order -> lse_i, loss_i
__global__ void __launch_bounds__(SM_NT)
sm_combine_kernel(const float *__restrict__ pm, const float *__restrict__ pl, const float *__restrict__ zt,
                  const int32_t *__restrict__ n_active_p, int M, int tile_rows, int B, int Bp, float *__restrict__ lse_out,
                  float *__restrict__ loss_i) {
    const int i = blockIdx.x * (SM_NT / 64) + (threadIdx.x >> 6);
    if (i >= B) return;
    const int lane = threadIdx.x & 63;
    const int n = sm_clamp_n(n_active_p, M);
    const int nt = (n + tile_rows - 1) / tile_rows;
    float m = -INFINITY, l = 0.f;
    for (int t = lane; t < nt; t += 64) {
        const float tm = pm[(int64_t)t * Bp + i], tl = pl[(int64_t)t * Bp + i];
        if (tm > m) { l *= __expf(m - tm); m = tm; }
        if (tm != -INFINITY) l += tl * __expf(tm - m);
    }
    const float wm = ks_wave_max(m);
    const float wl = ks_wave_sum(m == -INFINITY ? 0.f : l * __expf(m - wm));
    if (lane == 0) {
        const float lse = wm + __logf(wl);
        lse_out[i] = lse;
        loss_i[i] = lse - zt[i];
    }
}

// second pass: logit gradient g (exp(Zt[a][i] - lse_i) - [a == target_pos[i]]), zero for a >= n_active (up to the end of the
// class tile) and for i >= B (up to Bp).
template <class T>
__global__ void __launch_bounds__(T::NT)
sm_grad_kernel(const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, const int32_t *__restrict__ active_idx,
               const int32_t *__restrict__ n_active_p, const int32_t *__restrict__ target_pos, const float *__restrict__ lse,
               int B, int Bp, int D, int M, float scale, float g, uint16_t *__restrict__ dZ8) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::LDS_ELEMS];
    const int n_active = sm_clamp_n(n_active_p, M);
    const int tiles_s = (B + T::BN - 1) / T::BN;
    const int n_tiles = tiles_s * ((n_active + T::BM - 1) / T::BM);
    if ((int)blockIdx.x >= n_tiles) return;
    const int t = ks_xcd_remap(blockIdx.x, n_tiles);
    const int ts = t % tiles_s, tc = t / tiles_s;
    f32x16_t acc[T::FM][T::FN];
    sm_logits_tile<T>(X, W, active_idx, n_active, B, D, tc, ts, lds, acc);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / T::WAVES_N, wn = wave % T::WAVES_N;
    const int c0 = tc * T::BM + wm * T::WM; // first class row of this wave
#pragma unroll
    for (int fn = 0; fn < T::FN; ++fn) {
        const int i = ts * T::BN + wn * T::WN + fn * 32 + (lane & 31);
        const bool i_ok = i < B;
        const float ls = i_ok ? lse[i] : 0.f;
        const int tp = i_ok ? target_pos[i] : -1;
#pragma unroll
        for (int fm = 0; fm < T::FM; ++fm) {
            uint32_t pk[4][2];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                float d[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int c = c0 + sm_tile_row(fm, 2 * q + e, lane);
                    d[e] = (i_ok && c < n_active) ? g * (__expf(scale * acc[fm][fn][2 * q + e] - ls) - (c == tp ? 1.f : 0.f)) : 0.f;
                }
                pk[q >> 1][q & 1] = ks_pack_bf2(d[0], d[1]);
            }
            sm_store_block(pk, dZ8 + sm_dz_at(c0 + fm * 32 + 8 * (lane >> 5), i, Bp), Bp);
        }
    }
}

// ================================================================================================
// Stationary-operand versions of the two softmax passes (D <= 512): a workgroup keeps the MFMA
// fragments of 256 samples in registers and streams its share ("slab") of the active classes past them.
// The active classes are cut into G / tiles_s equal slabs (multiples of 32 rows), so the chip is loaded
// evenly whatever the active count; per-sample softmax statistics are carried in registers along the slab.
// ================================================================================================
// stage shape of the sweeps for a depth of KT k-tiles: two per stage where KT is even (half the barriers), twelve in flight
template <int KT, bool RAGGED> using SmSoe = KsSoe<KT, 96, KT % 2 == 0 ? 6 : 12, KT % 2 == 0 ? 2 : 1, RAGGED>;
#define KS_FUSED_MAX_SCALE 40.f // exp(-2 * scale) must stay a normal fp32 / bf16 number

// rows per slab for n64 = round_up(n_active, 64) rows and `slabs` slabs
__host__ __device__ __forceinline__ int sm_slab_rows(int n64, int slabs) {
    int h = (n64 + slabs - 1) / slabs;
    h = (h + 31) & ~31;
    return h < 32 ? 32 : h;
}

// Products kept between the two passes of a small problem (see sm_grad_kept_kernel), in the order in which the accumulators of
// a 32 x 32 block hold them: four pieces of 64 lanes x 16 bytes.  In 16-byte pieces: the first of class block cb, sample block sb.
__device__ __forceinline__ int64_t sm_kept_at(int cb, int sb, int Bp, int lane) { return ((int64_t)cb * (Bp >> 5) + sb) * 256 + lane; }

template <class CFG, bool KEEP>
__global__ void __launch_bounds__(512)
sm_stats_soe_kernel(const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, const int32_t *__restrict__ active_idx,
                    const int32_t *__restrict__ n_active_p, const int32_t *__restrict__ target_pos, int B, int Bp, int D, int M,
                    int tiles_s, float scale, float *__restrict__ pm, float *__restrict__ pl, float *__restrict__ zt,
                    float *__restrict__ kept) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[CFG::LDS_ELEMS + 2 * SM_LIDX_CAP]; // one array: see ks_gemm_soe.h
    int32_t *const s_lidx = (int32_t *)(lds + CFG::LDS_ELEMS);
    const int n = sm_clamp_n(n_active_p, M);
    const int n64 = (n + 63) & ~63;
    const int slabs = gridDim.x / tiles_s;
    const int h = sm_slab_rows(n64, slabs);
    const int id = ks_xcd_remap(blockIdx.x, gridDim.x);
    const int ts = id % tiles_s, slab = id / tiles_s;
    const int s0 = slab * h, s1 = (s0 + h < n64) ? s0 + h : n64;
    if (slab >= slabs || s0 >= s1) return;
    const int lane = threadIdx.x & 63;
    const int lim = n < s1 ? n : s1; // rows of this slab that are real classes
    const int i = ts * CFG::RES + ks_soe_col();
    const int tp = (i < B) ? target_pos[i] : -1;
    float m = -INFINITY, l = 0.f;
    // scale > 0 (checked by the host): statistics are carried on the raw products, m = max of acc,
    // l = sum exp(scale * (acc - m)) = sum exp2(fma(acc, k1, -k1 * m)); one fused multiply-add per element
    const float k1 = scale * 1.4426950408889634f;
    auto epi = [&](int c0, int rows_here, f32x16_t (&acc)[CFG::FM]) {
        if (KEEP && (i & ~31) < ((B + 63) & ~63)) { // (blocks of padding samples beyond what dW reads: nowhere)
            float4 *p = (float4 *)kept + sm_kept_at(c0 >> 5, i >> 5, Bp, lane);
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm)
                if (fm * 32 < rows_here) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        p[(int64_t)fm * Bp * 8 + q * 64] = make_float4(acc[fm][4 * q], acc[fm][4 * q + 1], acc[fm][4 * q + 2], acc[fm][4 * q + 3]);
                }
        }
        // the target logit of a sample whose label sits in this chunk (rare: a scan over this lane's rows)
        if (tp >= c0 && tp < c0 + CFG::CH && tp < lim) {
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (c0 + ks_soe_row(fm, r, lane) == tp) zt[i] = scale * acc[fm][r];
        }
        if (c0 + CFG::CH <= lim) { // every row of the chunk is a real class: no masks
            float cmax = acc[0][0];
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm)
#pragma unroll
                for (int r = 0; r < 16; ++r) cmax = fmaxf(cmax, acc[fm][r]);
            const float mn = fmaxf(m, cmax);
            const float off = -k1 * mn;
            float q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f; // four chains: the exponentials do not wait on one sum
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm)
#pragma unroll
                for (int r = 0; r < 16; r += 4) {
                    q0 += __builtin_amdgcn_exp2f(fmaf(acc[fm][r], k1, off));
                    q1 += __builtin_amdgcn_exp2f(fmaf(acc[fm][r + 1], k1, off));
                    q2 += __builtin_amdgcn_exp2f(fmaf(acc[fm][r + 2], k1, off));
                    q3 += __builtin_amdgcn_exp2f(fmaf(acc[fm][r + 3], k1, off));
                }
            l = l * __builtin_amdgcn_exp2f(k1 * (m - mn)) + ((q0 + q1) + (q2 + q3)); // m = -inf, l = 0 at the start
            m = mn;
        } else {
            float cmax = -INFINITY;
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (c0 + ks_soe_row(fm, r, lane) < lim) cmax = fmaxf(cmax, acc[fm][r]);
            if (cmax == -INFINITY) return; // no real class among this lane's rows of the chunk
            const float mn = fmaxf(m, cmax);
            const float off = -k1 * mn;
            float sum = 0.f;
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (c0 + ks_soe_row(fm, r, lane) < lim) sum += __builtin_amdgcn_exp2f(fmaf(acc[fm][r], k1, off));
            l = l * __builtin_amdgcn_exp2f(k1 * (m - mn)) + sum;
            m = mn;
        }
    };
    ks_soe_sweep<CFG>(X, D, ts * CFG::RES, B, W, D, active_idx, s0, s1, n, lds, epi, s_lidx, SM_LIDX_CAP);
    {
        // the two half-waves hold disjoint class rows of the same 32 samples
        const float mz = scale * m; // back to logit units
        const float mo = __shfl_xor(mz, 32, 64), lo = __shfl_xor(l, 32, 64);
        const float mm = fmaxf(mz, mo);
        const float ll = (mz == -INFINITY ? 0.f : l * __expf(mz - mm)) + (mo == -INFINITY ? 0.f : lo * __expf(mo - mm));
        if (lane < 32 && i < B) {
            pm[(int64_t)slab * Bp + i] = mm;
            pl[(int64_t)slab * Bp + i] = ll;
        }
    }
}

template <class CFG>
__global__ void __launch_bounds__(512)
sm_grad_soe_kernel(const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, const int32_t *__restrict__ active_idx,
                   const int32_t *__restrict__ n_active_p, const int32_t *__restrict__ target_pos,
                   const float *__restrict__ lse, int B, int Bp, int D, int M, int tiles_s, float scale, float g,
                   uint16_t *__restrict__ dZ8) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[CFG::LDS_ELEMS + 2 * SM_LIDX_CAP]; // one array: see ks_gemm_soe.h
    int32_t *const s_lidx = (int32_t *)(lds + CFG::LDS_ELEMS);
    const int n = sm_clamp_n(n_active_p, M);
    const int n64 = (n + 63) & ~63;
    const int slabs = gridDim.x / tiles_s;
    const int h = sm_slab_rows(n64, slabs);
    const int id = ks_xcd_remap(blockIdx.x, gridDim.x);
    const int ts = id % tiles_s, slab = id / tiles_s;
    const int s0 = slab * h, s1 = (s0 + h < n64) ? s0 + h : n64;
    if (slab >= slabs || s0 >= s1) return;
    const int i = ts * CFG::RES + ks_soe_col();
    const bool ok = i < B;
    const float ls = ok ? lse[i] : 0.f;
    const int tp = ok ? target_pos[i] : -1;
    // scale > 0 and g > 0 (checked by the host): g * exp(scale * acc - lse) = exp2(fma(acc, k1, k2)) with
    // k2 = log2(g) - lse * log2(e): one fused multiply-add and one exponential per element
    const float k1 = scale * 1.4426950408889634f;
    const float k2 = __log2f(g) - ls * 1.4426950408889634f;
    const bool samples_ok = (ts + 1) * CFG::RES <= B;
    auto epi = [&](int c0, int rows_here, f32x16_t (&acc)[CFG::FM]) {
        const int lane = threadIdx.x & 63;
        const bool plain = samples_ok && c0 + CFG::CH <= n; // no row or column of this chunk needs masking
        const int tq = tp - c0 - 4 * (lane >> 5);           // the own class's accumulator element: fm * 32 + 8 * (r >> 2) + (r & 3) == tq
        const int lq = ok ? n - c0 - 4 * (lane >> 5) : 0;           // the first of its elements to mask
        const bool any_target = __any(tp >= c0 && tp < c0 + CFG::CH);
        if (!plain) {
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (fm * 32 + 8 * (r >> 2) + (r & 3) >= lq) acc[fm][r] = -INFINITY; // its exponential is 0
        }
        uint16_t *p = dZ8 + sm_dz_at(c0 + 8 * (lane >> 5), i, Bp);
#pragma unroll
        for (int fm = 0; fm < CFG::FM; ++fm) {
            uint32_t pk[4][2];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                float d[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) d[e] = __builtin_amdgcn_exp2f(fmaf(acc[fm][2 * q + e], k1, k2));
                if (any_target) {
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        if (fm * 32 + 8 * (q >> 1) + 2 * (q & 1) + e == tq) d[e] -= g;
                }
                pk[q >> 1][q & 1] = ks_pack_bf2(d[0], d[1]);
            }
            if (fm * 32 < rows_here) sm_store_block(pk, p + (int64_t)fm * 4 * Bp * 8, Bp);
        }
    };
    ks_soe_sweep<CFG, 2 * CFG::FM>(X, D, ts * CFG::RES, B, W, D, active_idx, s0, s1, n, lds, epi, s_lidx, SM_LIDX_CAP);
}


// Small problems (sm_kept_bytes): the second sweep and the merge of the slabs' statistics before it as one pass over the products, which the
// first sweep has kept (fp32, as they stood in its accumulators: the same gradient bit for bit but for the order of the merge).
// A workgroup has 32 samples and takes every gridDim.y-th group of four class blocks; it merges its samples' statistics itself,
// while its first block is on the way.  Blocks of padding samples are left out but for the one that completes dW's k-tile of 64
// (12,000 classes x 512, batch 33: 47.9 -> 44.3 us; 8,192 x 320: 39.3 -> 35.4).  (2,297 classes x 320, batch 333: merge and sweep 3.9 + 9.2 us, this 6.3.)
__global__ void __launch_bounds__(SM_NT)
sm_grad_kept_kernel(const float *__restrict__ kept, const float *__restrict__ pm, const float *__restrict__ pl, const float *__restrict__ zt,
                    const int32_t *__restrict__ n_active_p, const int32_t *__restrict__ target_pos, int B, int Bp, int M, int slabs,
                    float scale, float g, float *__restrict__ loss_i, uint16_t *__restrict__ dZ8) {
    constexpr int PARTS = SM_NT / 32;
    __shared__ float s_m[PARTS][32], s_l[PARTS][32];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sb = blockIdx.x, cb0 = blockIdx.y * 4 + wave;
    float4 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    auto fetch = [&](int cb) __attribute__((always_inline)) {
        const float4 *p = (const float4 *)kept + sm_kept_at(cb, sb, Bp, lane);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = p[q * 64];
    };
    if (cb0 * 32 < M) fetch(cb0); // (the array has whole blocks for M rows)
    const int n = sm_clamp_n(n_active_p, M);
    const int n64 = (n + 63) & ~63, h = sm_slab_rows(n64, slabs);
    const int j = threadIdx.x & 31, part = threadIdx.x >> 5;
    {
        const int i = sb * 32 + j;
        float m = -INFINITY, l = 0.f;
        for (int t0 = part; t0 * h < n64; t0 += 8 * PARTS) { // (slabs that hold rows; i < Bp)
            float tm[8], tl[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int t = t0 + u * PARTS;
                const bool in = t * h < n64 && i < B;
                tm[u] = in ? pm[(int64_t)t * Bp + i] : -INFINITY;
                tl[u] = in ? pl[(int64_t)t * Bp + i] : 0.f;
            }
            float mm = m;
#pragma unroll
            for (int u = 0; u < 8; ++u) mm = fmaxf(mm, tm[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u) tl[u] = tm[u] != -INFINITY ? tl[u] * __expf(tm[u] - mm) : 0.f;
            if (mm != -INFINITY) l = l * __expf(m - mm) + (((tl[0] + tl[1]) + (tl[2] + tl[3])) + ((tl[4] + tl[5]) + (tl[6] + tl[7])));
            m = mm; // (m = -inf, l = 0 at the start)
        }
        s_m[part][j] = m;
        s_l[part][j] = l;
    }
    __syncthreads();
    const int i = sb * 32 + (lane & 31);
    const bool ok = i < B;
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) m = fmaxf(m, s_m[p][lane & 31]);
    float lp[PARTS];
#pragma unroll
    for (int p = 0; p < PARTS; ++p) lp[p] = s_m[p][lane & 31] != -INFINITY ? s_l[p][lane & 31] * __expf(s_m[p][lane & 31] - m) : 0.f;
#pragma unroll
    for (int o = PARTS / 2; o > 0; o >>= 1) // a tree: as close to the exact sum as the merge by a wavefront
#pragma unroll
        for (int p = 0; p < o; ++p) lp[p] += lp[p + o];
    l = lp[0];
    const float lse = m + __logf(l);
    const int tp = ok ? target_pos[i] : -1;
    if (blockIdx.y == 0 && threadIdx.x < 32 && ok) loss_i[i] = lse - zt[i];
    // scale > 0 and g > 0 (checked by the host), as in sm_grad_soe_kernel
    const float k1 = scale * 1.4426950408889634f;
    const float k2 = __log2f(g) - (ok ? lse : 0.f) * 1.4426950408889634f;
    for (int cb = cb0; cb * 32 < n64; cb += gridDim.y * 4) {
        const int c0 = cb * 32, tq = tp - c0 - 4 * (lane >> 5), lq = ok ? n - c0 - 4 * (lane >> 5) : 0;
        uint32_t pk[4][2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float d[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                d[e] = 8 * q + e >= lq ? 0.f : __builtin_amdgcn_exp2f(fmaf(d[e], k1, k2));
                if (8 * q + e == tq) d[e] -= g;
            }
            pk[q][0] = ks_pack_bf2(d[0], d[1]);
            pk[q][1] = ks_pack_bf2(d[2], d[3]);
        }
        const int next = cb + gridDim.y * 4;
        if (next * 32 < n64) fetch(next);
        sm_store_block(pk, dZ8 + sm_dz_at(c0 + 8 * (lane >> 5), i, Bp), Bp);
    }
}

// ------------------------------------------------------------------------------------------------
// One-sweep variant for rows of norm <= 1 (the paper normalises W and X, section 3.2): every logit
// lies in [-scale, scale], so the softmax can be evaluated against the fixed reference `scale` and no
// statistics pass is needed.  The sweep writes E[a][i] = exp(z_ia - scale) (bf16, transposed, zero in the
// padding and at the sample's own class) and per-slab sums of the stored (rounded) E; sm_combine then forms
// sum_i = sum_a E_ia and the loss.  Column i of the gradient, (P_ia - [a = target_i]) * sum_i, is the stored column
// and one entry more, E_t - sum_i at the own class, which never goes into the stored array: its term of dX is
// a partial product of its own, and dW puts it into its tile in LDS.  The factor g / sum_i that is still missing is
// applied where it is cheap: on the rows of dX after the contraction over classes, and on the rows of X
// (X2 = X / sum_i, bf16) before the contraction over samples.
// The reference only shifts the exponent range: results are the same function of the inputs as long as no
// exponential overflows and not all of a sample's vanish, which the combine kernel checks.
// ------------------------------------------------------------------------------------------------
// The sweep runs on the eight-wavefront engine (ks_gemm_soe.h): wavefront w owns samples [32 w, 32 w + 32) of the
// tile and two wavefronts share a SIMD, so the exponentials and stores of one overlap with the MFMAs of the other.
// The sums of the stored (rounded) values come from the matrix pipe: a product with a block of ones on the packed values.
template <class CFG>
__global__ void __launch_bounds__(512)
sm_fused_soe_kernel(const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, const int32_t *__restrict__ active_idx,
                     const int32_t *__restrict__ n_active_p, const int32_t *__restrict__ target_pos, int B, int Bp, int D, int M,
                     int tiles_s, float scale, float *__restrict__ pl, float *__restrict__ pl_others, uint16_t *__restrict__ dZ8) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[CFG::LDS_ELEMS + 2 * SM_LIDX_CAP]; // one array: see ks_gemm_soe.h
    int32_t *const s_lidx = (int32_t *)(lds + CFG::LDS_ELEMS);
    const int n = sm_clamp_n(n_active_p, M);
    const int n64 = (n + 63) & ~63;
    const int slabs = gridDim.x / tiles_s;
    const int h = sm_slab_rows(n64, slabs);
    const int id = ks_xcd_remap(blockIdx.x, gridDim.x);
    const int ts = id % tiles_s, slab = id / tiles_s;
    const int s0 = slab * h, s1 = (s0 + h < n64) ? s0 + h : n64;
    if (slab >= slabs || s0 >= s1) return;
    const int lim = n < s1 ? n : s1; // rows of this slab that are real classes
    const float k1 = scale * 1.4426950408889634f; // exp(scale * acc - scale) = exp2(fma(acc, k1, -k1))
    const bool samples_ok = (ts + 1) * CFG::RES <= B;
    const int i = ts * CFG::RES + ks_soe_col();
    const bool ok = i < B;
    const int my_tp = ok ? target_pos[i] : -1; // position of this lane's sample's class in the active list
    // For the loss: this lane's sum of the UNROUNDED exponentials of its sample over its rows, the sample's own class
    // left out (the combine step adds that one from an fp32 dot product).  The sums of the stored, rounded values
    // (`pl`) are what the gradient columns must add up to; for the loss of a confident sample they would carry the
    // bf16 rounding of its strongest competitor, 2^-9 relative.  The own class is left out of those too, and stored as 0,
    // which it stays (see sm_combine).
    float others = 0.f;
    f32x4_t rounded = {0.f, 0.f, 0.f, 0.f}; // every element: the sum of the values that this lane has stored
    auto epi = [&](int c0, int rows_here, f32x16_t (&acc)[CFG::FM]) {
        const int lane = threadIdx.x & 63;
        const bool plain = samples_ok && c0 + CFG::CH <= lim; // no row or column of this chunk needs masking
        const int tl = my_tp - c0;                             // the own class's row in this chunk, if in [0, CH)
        uint16_t *p = dZ8 + sm_dz_at(c0 + 8 * (lane >> 5), i, Bp); // (i < Bp: whole tiles exist)
        typedef short s16x4_t __attribute__((ext_vector_type(4)));
        const s16x4_t ones = {0x3F80, 0x3F80, 0x3F80, 0x3F80}; // bf16
        float c4[4] = {0.f, 0.f, 0.f, 0.f}; // four chains: the additions do not wait on one sum
        if (!plain || __any(tl >= 0 && tl < CFG::CH)) { // rows or samples to mask, or some sample of this wavefront has its class here
            // accumulator element (fm, r) is row fm * 32 + 8 * (r >> 2) + (r & 3) + 4 * (lane >> 5)
            const int tq = tl - 4 * (lane >> 5), lq = ok ? lim - c0 - 4 * (lane >> 5) : 0;
#pragma unroll
            for (int fm = 0; fm < CFG::FM; ++fm)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int e = fm * 32 + 8 * (r >> 2) + (r & 3);
                    if (e == tq || e >= lq) acc[fm][r] = -INFINITY; // its exponential is 0
                }
        }
#pragma unroll
        for (int fm = 0; fm < CFG::FM; ++fm) {
            uint32_t pk[4][2];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                float d[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    d[e] = __builtin_amdgcn_exp2f(fmaf(acc[fm][2 * q + e], k1, -k1));
                    c4[2 * (q & 1) + e] += d[e];
                }
                pk[q >> 1][q & 1] = ks_pack_bf2(d[0], d[1]);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) // (sixteen 4 x 4 products side by side: a lane's four k's of its own column)
                rounded = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4_t, (ks_u32x2){pk[g][0], pk[g][1]}), rounded, 0, 0, 0);
            if (fm * 32 < rows_here) sm_store_block(pk, p + (int64_t)fm * 4 * Bp * 8, Bp);
            __builtin_amdgcn_sched_barrier(0); // one block's values at a time: the sweep leaves few registers
        }
        others += (c4[0] + c4[1]) + (c4[2] + c4[3]);
    };
    ks_soe_sweep<CFG, 2 * CFG::FM>(X, D, ts * CFG::RES, B, W, D, active_idx, s0, s1, n, lds, epi, s_lidx, SM_LIDX_CAP);
    others += __shfl_xor(others, 32, 64); // the two lanes of a sample hold different rows
    const float stored = rounded[0] + __shfl_xor(rounded[0], 32, 64);
    if ((threadIdx.x & 63) < 32 && ok) {
        pl[(int64_t)slab * Bp + i] = stored;
        pl_others[(int64_t)slab * Bp + i] = others;
    }
}

// Combine step of the one-sweep variant, per sample: the sum of the slab sums; the target logit as an fp32 dot product of
// the two bf16 rows and with it the target's exponential E_t and the loss; the reciprocal sum for dX; the scaled row of X2.
// The column of the logit gradient is (P - onehot) * sum when the target's entry, which the sweep has stored as 0, is
// E_t - sum = -(sum of the others): so it sums to zero and P_t - 1 carries no cancellation.  That entry does not go into the
// stored column, which the dX launch is reading: its term of dX, entry times the class's row, becomes one more partial product
// (fp32, where the other entries are rounded to bf16), and the dW kernel puts the rounded entry into its tile in LDS.  So the
// step needs no launch of its own here, only blocks beside the dX tiles (before: a kernel between the sweep and dX, 5.2 to
// 7.9 us of every step).
#define SM_CF_NT 256
// The softmax split over the nodes of the model-parallel layer (Section 3.1 steps 3-5) runs the same kernels in two
// calls with an exchange of the per-sample statistics in between:
#define SM_WHOLE 0  /* one GPU owns all classes: statistics and gradient in one go */
#define SM_EXPORT 1 /* first call: this node's statistics go out, nothing is normalised yet */
#define SM_IMPORT 2 /* second call: the statistics combined over all nodes come in */
struct SmSplitIO {
    float *row_max, *row_sum, *tz_out;    // SM_EXPORT
    const float *gmax, *gsum, *gtz;       // SM_IMPORT
};
struct SmCombine {
    int blocks;             // workgroups that do it (0: nothing to do), SM_CF_FEW or SM_CF_MANY samples each
    int many;
    const float *pl, *pl_others; // the sweep's slab sums
    int slabs, D;                // D: 128, 256 or 512
    const int32_t *target_pos;
    const uint16_t *X;
    float scale;
    float *inv_sum, *loss_i;
    uint16_t *X2;
    float *extra;           // [B][D]: the targets' terms of dX (a further partial product)
    int32_t *cell_pos;      // [Bp]: where dW's target entry goes (-1: nowhere) ...
    uint32_t *cell;         // [Bp]: ... and its bf16 value
    int32_t *dev_status;
    int mode;
    SmSplitIO io;
};
#define SM_CF_FEW 8   /* the kernel is a chain of dependent round trips: spread over many compute units where there is room */
#define SM_CF_MANY 32
// Workgroup blk of job.blocks.  sh: 2 * NT + 4 * SPB floats of LDS.
template <int NT, int SPB>
__device__ __forceinline__ void sm_combine(const SmCombine &job, int blk, const int32_t *__restrict__ n_active_p, int M, int B, int Bp,
                                           const int32_t *__restrict__ active_idx, const uint16_t *__restrict__ W, float *sh) {
    constexpr int PARTS = NT / SPB;                      // threads per sample: each takes a share of the slab sums
    constexpr int U = SPB * 64 >= NT ? SPB * 64 / NT : 1; // 16-byte pieces of rows per thread, at D = 512
    const int D = job.D, per_row = D / 8;
    const int rows = B - blk * SPB < SPB ? B - blk * SPB : SPB, total = rows * per_row;
    const int64_t first = (int64_t)blk * SPB * D; // the block's rows are contiguous
    float *const s_inv = sh + 2 * NT, *const s_cell = s_inv + SPB, *const s_dot = s_cell + SPB;
    // pieces of the rows of X and of the samples' classes, the slab sums: requested before anything is waited for
    int tp[U], cls[U];
    uint4 x[U], w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int q = u * NT + threadIdx.x;
        tp[u] = q < total ? job.target_pos[blk * SPB + q / per_row] : -1;
        x[u] = q < total ? *(const uint4 *)(job.X + first + (int64_t)q * 8) : make_uint4(0u, 0u, 0u, 0u);
    }
    const int j = threadIdx.x % SPB, gq = threadIdx.x / SPB, i = blk * SPB + j;
    const int n = sm_clamp_n(n_active_p, M);
    const int n64 = (n + 63) & ~63, h = sm_slab_rows(n64, job.slabs);
    float part = 0.f, oth = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) cls[u] = tp[u] >= 0 && tp[u] < n ? active_idx[tp[u]] : -1;
    if (i < B && job.mode != SM_IMPORT) {
        for (int t0 = gq; t0 * h < n64; t0 += 4 * PARTS) { // (slabs that hold rows)
            float v[4], o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = (t0 + PARTS * q) * h < n64;
                v[q] = in ? job.pl[(int64_t)(t0 + PARTS * q) * Bp + i] : 0.f;
                o[q] = in ? job.pl_others[(int64_t)(t0 + PARTS * q) * Bp + i] : 0.f;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                part += v[q];
                oth += o[q];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        w[u] = cls[u] >= 0 ? *(const uint4 *)(W + (int64_t)cls[u] * D + (u * NT + threadIdx.x) % per_row * 8) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t xs[4] = {x[u].x, x[u].y, x[u].z, x[u].w}, ws[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dot = fmaf(ks_bf2f(xs[e] & 0xFFFFu), ks_bf2f(ws[e] & 0xFFFFu), dot);
            dot = fmaf(ks_bf2f(xs[e] >> 16), ks_bf2f(ws[e] >> 16), dot);
        }
        for (int o = per_row / 2; o > 0; o >>= 1) dot += __shfl_xor(dot, o, 64); // (a row's pieces are neighbouring lanes)
        const int q = u * NT + threadIdx.x;
        if (q < total && q % per_row == 0) {
            s_dot[q / per_row] = dot;
            s_cell[q / per_row] = cls[u] >= 0 ? 1.f : 0.f; // (for now: whether the sample's class is here)
        }
    }
    sh[threadIdx.x] = part;
    sh[NT + threadIdx.x] = oth;
    __syncthreads();
    if ((int)threadIdx.x < SPB && i < B) {
        float inv = 0.f, cell = 0.f, others = 0.f;
        oth = 0.f;
        for (int q = 0; q < PARTS; ++q) { // a fixed order
            others += sh[q * SPB + j];
            oth += sh[NT + q * SPB + j];
        }
        const bool owned = s_cell[j] != 0.f; // (one GPU: always, unless the list is broken; split over nodes: this node's class)
        const float z_t = job.scale * s_dot[j];
        const float e_t = __expf(z_t - job.scale);
        if (job.mode == SM_IMPORT) {
            // the sum over the classes of all nodes, brought to this kernel's reference `scale`
            const float S = job.io.gsum[i] * __expf(job.io.gmax[i] - job.scale);
            if (!(S > 0.f) || !(S < INFINITY)) ks_flag(job.dev_status, KS_DEV_RANGE);
            job.loss_i[i] = (job.io.gmax[i] + __logf(job.io.gsum[i])) - job.io.gtz[i];
            inv = 1.f / S;
            cell = e_t - S; // (P_t - 1) * S
        } else {
            const float sum = owned ? others + e_t : others; // (the sweep leaves the sample's own class out)
            if (job.mode == SM_EXPORT) {
                job.io.row_max[i] = job.scale;
                job.io.row_sum[i] = sum;
                job.io.tz_out[i] = owned ? z_t : 0.f;
            } else {
                if (!(sum > 0.f) || !(sum < INFINITY)) ks_flag(job.dev_status, KS_DEV_RANGE);
                // loss = log(1 + (unrounded exponentials of the other classes) / E_t): no difference of nearly
                // equal numbers, and no bf16 rounding in it
                const float ratio = oth / e_t;
                job.loss_i[i] = (owned && ratio < 1e30f) ? log1pf(ratio) : (job.scale + __logf(sum)) - z_t;
                inv = 1.f / sum;
                cell = -others;
            }
        }
        if (job.mode != SM_EXPORT) {
            job.inv_sum[i] = inv;
            job.cell_pos[i] = owned ? job.target_pos[i] : -1;
            job.cell[i] = ks_f2bf(cell);
        }
        s_inv[j] = inv;
        s_cell[j] = owned ? cell : 0.f;
    }
    if (job.mode == SM_EXPORT) return; // nothing is normalised before the nodes have exchanged their sums
    __syncthreads();
    auto scaled = [](uint32_t v, float f) __attribute__((always_inline)) { return ks_pack_bf2(ks_bf2f(v & 0xFFFFu) * f, ks_bf2f(v >> 16) * f); };
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int q = u * NT + threadIdx.x;
        if (q < total) {
            const float f = s_inv[q / per_row], c = s_cell[q / per_row];
            *(uint4 *)(job.X2 + first + (int64_t)q * 8) = make_uint4(scaled(x[u].x, f), scaled(x[u].y, f), scaled(x[u].z, f), scaled(x[u].w, f));
            float4 *e = (float4 *)(job.extra + first + (int64_t)q * 8);
            e[0] = make_float4(c * ks_bf2f(w[u].x & 0xFFFFu), c * ks_bf2f(w[u].x >> 16), c * ks_bf2f(w[u].y & 0xFFFFu), c * ks_bf2f(w[u].y >> 16));
            e[1] = make_float4(c * ks_bf2f(w[u].z & 0xFFFFu), c * ks_bf2f(w[u].z >> 16), c * ks_bf2f(w[u].w & 0xFFFFu), c * ks_bf2f(w[u].w >> 16));
        }
    }
}
// the same as a launch of its own: the first call of a softmax split over nodes ends with it
__global__ void __launch_bounds__(SM_CF_NT)
sm_combine_fused_kernel(SmCombine job, const int32_t *__restrict__ n_active_p, int M, int B, int Bp, const int32_t *__restrict__ active_idx,
                        const uint16_t *__restrict__ W) {
    __shared__ float sh[2 * SM_CF_NT + 4 * SM_CF_FEW];
    sm_combine<SM_CF_NT, SM_CF_FEW>(job, blockIdx.x, n_active_p, M, B, Bp, active_idx, W, sh);
}

// one wavefront per sample: merge the per-slab (max, sum) pairs in slab order -> lse_i, loss_i
__global__ void __launch_bounds__(SM_NT)
sm_combine_soe_kernel(const float *__restrict__ pm, const float *__restrict__ pl, const float *__restrict__ zt,
                      const int32_t *__restrict__ n_active_p, int M, int slabs, int B, int Bp, float *__restrict__ lse_out,
                      float *__restrict__ loss_i) {
    const int i = blockIdx.x * (SM_NT / 64) + (threadIdx.x >> 6);
    if (i >= B) return;
    const int lane = threadIdx.x & 63;
    const int n = sm_clamp_n(n_active_p, M);
    const int n64 = (n + 63) & ~63;
    const int h = sm_slab_rows(n64, slabs);
    const int nt = (n64 + h - 1) / h;
    float m = -INFINITY, l = 0.f;
    for (int t = lane; t < nt; t += 64) {
        const float tm = pm[(int64_t)t * Bp + i], tl = pl[(int64_t)t * Bp + i];
        if (tm > m) { l *= __expf(m - tm); m = tm; }
        if (tm != -INFINITY) l += tl * __expf(tm - m);
    }
    const float wm = ks_wave_max(m);
    const float wl = ks_wave_sum(m == -INFINITY ? 0.f : l * __expf(m - wm));
    if (lane == 0) {
        const float lse = wm + __logf(wl);
        lse_out[i] = lse;
        loss_i[i] = lse - zt[i];
    }
}

// dX partials on the asynchronous engine: P[s][i][d] = sum_{a in share s} dZ[a][i] * W[active[a]][d].
// dZ8 as stored is the operand in blocks of eight k's (k = a); the weight rows, fetched through the index list, are k-major.
template <class T>
__global__ void __launch_bounds__(T::NT)
dx_partial_async_kernel(const uint16_t *__restrict__ dZ8, int Bp, const uint16_t *__restrict__ W,
                        const int32_t *__restrict__ active_idx, const int32_t *__restrict__ n_active_p, int B, int D, int M,
                        int S, float *__restrict__ part, SmCombine comb, KsSelNext next) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::LDS_ELEMS];
    __shared__ int32_t s_idx[DxIdx<T>::CAP];
    const int bid = (int)blockIdx.x - comb.blocks;
    if (bid < 0) { // blocks before the tiles: the one-sweep softmax's combine step
        if (comb.many) sm_combine<T::NT, SM_CF_MANY>(comb, (int)blockIdx.x, n_active_p, M, B, Bp, active_idx, W, (float *)lds);
        else sm_combine<T::NT, SM_CF_FEW>(comb, (int)blockIdx.x, n_active_p, M, B, Bp, active_idx, W, (float *)lds);
        return;
    }
    const int n_active = sm_clamp_n(n_active_p, M);
    const int tiles_m = (B + T::BM - 1) / T::BM, tiles_n = (D + T::BN - 1) / T::BN;
    const int n_tiles = tiles_m * tiles_n;
    if (bid >= n_tiles * S) { // blocks behind the tiles: the next batch's candidates are staged (if asked for)
        ks_sel_next_fetch<T::NT>(next, bid - n_tiles * S);
        return;
    }
    const int L = ks_xcd_remap(bid, n_tiles * S);
    const int s = L / n_tiles, t = L % n_tiles;
    const int tm = t % tiles_m, tn = t / tiles_m;
    const int nk = (n_active + 63) / 64;
    const int per = (nk + S - 1) / S;
    const int kt0 = s * per, kt1 = (kt0 + per < nk) ? kt0 + per : nk;
    f32x16_t acc[T::FM][T::FN];
    ks_a_clear<T>(acc);
    if (kt0 < kt1) {
        // gather list of this share, staged in LDS (the host sizes S so that a share fits), clamped at the end:
        // rows at or beyond n_active meet zeros of dZ8
        for (int e = threadIdx.x; e < (kt1 - kt0) * 64 && e < DxIdx<T>::CAP; e += T::NT) {
            int k = kt0 * 64 + e;
            if (k >= n_active) k = n_active - 1;
            s_idx[e] = active_idx[k];
        }
        __syncthreads();
        KsAK8<T::BM, T::NW> ar;
        KsAKmaj<T::BN, T::NW> br;
        ar.init(dZ8, Bp, tm * T::BM); // (Bp is a multiple of the tile)
        br.init(W, D, s_idx, tn * T::BN, D, kt1 * 64, kt0 * 64);
        ks_a_mainloop<T, KS_K8, KS_KMAJ>(ar, br, kt0, kt1, lds, acc);
    }
    // row-wise through LDS (the main loop has ended with a barrier): 16-byte pieces of whole rows, a quarter of the
    // store instructions of an element-wise hand-out
    float *out = part + (int64_t)s * B * D;
    typedef KsASlab<T> SL;
    float *st = (float *)lds;
    for (int p = 0; p < T::WAVES_M; ++p) {
        ks_a_stage_slab<T>(acc, st, p);
        __syncthreads();
        constexpr int PER = SL::ROWS * SL::QUADS / T::NT;
        static_assert(SL::ROWS * SL::QUADS % T::NT == 0, "slab shape");
#pragma unroll 4
        for (int q0 = 0; q0 < PER; ++q0) {
            const int q = q0 * T::NT + threadIdx.x;
            const int row = q / SL::QUADS, quad = q % SL::QUADS;
            const int i = tm * T::BM + p * SL::ROWS + row, d = tn * T::BN + quad * 4;
            if (i < B && d < D) *(float4 *)(out + (int64_t)i * D + d) = ks_a_slab_quad<T>(st, row, quad); // D % 4 == 0
        }
        __syncthreads();
    }
}

// dW_active[a][d] = scale * sum_i dZ[a][i] * X[i][d] on the asynchronous engine (X k-major, k = i).
// The grid is sized for M rows, so with fewer active rows part of the chip would idle; the last
// DW_REDUCE_BLOCKS blocks of the grid therefore do a job that is due anyway and does not depend on this
// kernel: the sum of the dX partial products of the kernel before (with the per-sample factor, if any) and
// the batch mean of the losses.  They land on the compute units the tiles leave free.
#define DW_REDUCE_BLOCKS 128
struct DxReduceJob {
    const float *part; // [S][B * D] partial sums
    int S;
    int64_t BD;
    float scale;
    const float *row_factor; // [B] or nullptr
    float *dX;
    const float *loss_i;
    float *loss_mean;
};
// The weight update of Section 3.1 step 6 done where the gradient is produced: the tile that has just computed a
// block of dW_active adds alpha times it to the fp32 rows of the active classes and refreshes their 16-bit copy,
// so the gradient never travels to memory and back (same arithmetic as the stand-alone update: one fused
// multiply-add per element on the stored fp32 value of the gradient).  Wm == nullptr: no update.
struct DwUpdate {
    float *Wm;
    uint16_t *Wb;
    const int32_t *idx;
    float alpha;
};
// Entries of the logit gradient that are not in the stored array (its place holds 0): sample i has the bf16 value val[i] in row
// pos[i] (-1: none).  pos == nullptr: the array is complete.
struct DwCells {
    const int32_t *pos;
    const uint32_t *val;
};
// Shape of the dW tiles for n_active rows on a chip of n_cu compute units (one tile per compute unit at a time); the launch
// has workgroups for tiles_max of them.  A tile is a chain -- its k-tiles, then its part of the update, round trip after round
// trip -- so with few rows the smallest tiles that still fit the chip in one round are the fastest; tall tiles load the X panel
// and a wide tile the dZ8 panel less often, which counts once every compute unit has a tile.  Estimated time = rounds x cost
// of a lone tile x (1 + share of the compute units at work: the memory is shared); the smallest wins, ties to the larger tile.
// The costs are fitted to whole calls with each shape forced, at 1,700 sizes of D = 64 to 512, B = 33 to 2,048, A = 600 to
// 110,000: the call with the shape chosen is 0.2 % slower than with the best one on average, 8 % at most (the batch makes no
// difference to the choice, and near ties may go either way).  us, 256 x 256, 192 x 256, 128 x 256, 128 x 128, 64 x 128: dW and
// update, list of A classes: D = 128, B = 64, A = 600: 16.3, 11.2, 8.4, 5.9, 5.1; D = 320, B = 333, A = 3,001: 21.3, 16.6, 12.4,
// 9.0, 7.8; D = 512, B = 1,024, A = 4,725: 36.5, 29.1, 24.0, 21.6, 25.2; A = 17,425: 48.9, 40.0, 51.0, 51.6, 58.7; A = 32,374:
// 54.0, 58.8, 57.8, 67.3, 91.0.  Whole calls: D = 512, B = 2,048, A = 6,529: 123.5, 109.3, 100.8, 90.7, 109.4; D = 256, B = 1,024,
// A = 6,529: 72.5, 62.2, 57.2, 52.1, 47.5; D = 512, B = 64, A = 15,391: 44.1, 40.4, 43.8, 45.1, 44.0.  (64 x 256: never ahead of
// 128 x 128.)
enum { DW_KINDS = 5 };
__device__ __forceinline__ int dw_tile_kind(int n_active, int D, int n_cu, int tiles_max) {
    const int rows[DW_KINDS] = {TileDw::BM, TileDw192::BM, TileDw128::BM, TileDw128n::BM, TileDw64n::BM};
    const int cols[DW_KINDS] = {TileDw::BN, TileDw192::BN, TileDw128::BN, TileDw128n::BN, TileDw64n::BN};
    const float cost[DW_KINDS] = {31.5f, 21.24f, 18.0f, 13.78f, 10.57f};
    const float per_cu = 1.f / (float)n_cu;
    int best = 0;
    float best_t = INFINITY;
#pragma unroll
    for (int k = 0; k < DW_KINDS; ++k) {
        const int tiles = ((D + cols[k] - 1) / cols[k]) * ((n_active + rows[k] - 1) / rows[k]);
        const float share = (float)tiles * per_cu;
        const float t = ceilf(share) * cost[k] * (1.f + 0.98f * fminf(share, 1.f));
        if (t < best_t && tiles <= tiles_max) { best_t = t; best = k; }
    }
    return best;
}

// LDS of the launch: a tile's stages, its rows' classes and its k-tiles' cells, or the bitmap of the next batch's selection
#define DW_CELL_SLOTS 4 /* k-tiles whose cells lie in LDS */
constexpr int DW_TILE_ELEMS = TileDw::LDS_ELEMS + 2 * (TileDw::BM + DW_CELL_SLOTS * 128);
constexpr int DW_LDS_ELEMS = DW_TILE_ELEMS > 2 * SEL1_LDS_WORDS ? DW_TILE_ELEMS : 2 * SEL1_LDS_WORDS;
template <class T, bool CELLS>
__device__ __forceinline__ void dw_tile(int bid, uint16_t *lds, const uint16_t *__restrict__ dZ8, const uint16_t *__restrict__ X, int B,
                                        int Bp, int n_active, int D, int64_t Mp, float scale, float *__restrict__ dW,
                                        const DwUpdate &up, const DwCells &cells);

template <bool CELLS>
__global__ void __launch_bounds__(TileDw::NT)
dw_async_kernel(const uint16_t *__restrict__ dZ8, const uint16_t *__restrict__ X, int B, int Bp,
                const int32_t *__restrict__ n_active_p, int D, int M, int64_t Mp, float scale, float *__restrict__ dW,
                int tiles_max, int n_cu, DxReduceJob job, DwUpdate up, DwCells cells, KsSelNext next) {
    typedef TileDw T;
    __shared__ __attribute__((aligned(16))) uint16_t lds[DW_LDS_ELEMS];
    // The first next.nsel workgroups select the NEXT batch's active classes (Algorithm 1 needs only its labels): with a
    // few hundred tiles this launch leaves compute units idle, and being first they start at once.
    const int bid = (int)blockIdx.x - next.nsel;
    if (bid < 0) {
        ks_sel_next_select<T::NT>(next, (uint32_t *)lds, (int)blockIdx.x);
        return;
    }
    if (bid >= tiles_max) { // reduction blocks
        const int rb = bid - tiles_max, nrb = (int)gridDim.x - next.nsel - tiles_max;
        for (int64_t e = ((int64_t)rb * T::NT + threadIdx.x) * 4; e < job.BD; e += (int64_t)nrb * T::NT * 4) {
            const float f = job.row_factor ? job.scale * job.row_factor[e / D] : job.scale;
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int s0 = 0; s0 < job.S; s0 += 8) { // eight loads in flight, added in order
                float4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    v[u] = s0 + u < job.S ? *(const float4 *)(job.part + (int64_t)(s0 + u) * job.BD + e) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int u = 0; u < 8; ++u) { acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w; }
            }
            *(float4 *)(job.dX + e) = make_float4(f * acc.x, f * acc.y, f * acc.z, f * acc.w);
        }
        if (rb == nrb - 1) { // thread t takes samples t, t + NT, ..., then a tree: a fixed order
            float *sh = (float *)lds;
            float sum = 0.f;
            for (int i = threadIdx.x; i < B; i += T::NT) sum += job.loss_i[i];
            sh[threadIdx.x] = sum;
            __syncthreads();
            for (int o = T::NT / 2; o > 0; o >>= 1) {
                if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
                __syncthreads();
            }
            if (threadIdx.x == 0) *job.loss_mean = sh[0] / (float)B;
        }
        return;
    }
    const int n_active = sm_clamp_n(n_active_p, M);
    const int kind = dw_tile_kind(n_active, D, n_cu, tiles_max);
#define DW_TILE(T) dw_tile<T, CELLS>(bid, lds, dZ8, X, B, Bp, n_active, D, Mp, scale, dW, up, cells)
    if (kind == 0) DW_TILE(TileDw);
    else if (kind == 1) DW_TILE(TileDw192);
    else if (kind == 2) DW_TILE(TileDw128);
    else if (kind == 3) DW_TILE(TileDw128n);
    else DW_TILE(TileDw64n);
#undef DW_TILE
}

template <class T, bool CELLS>
__device__ __forceinline__ void dw_tile(int bid, uint16_t *lds, const uint16_t *__restrict__ dZ8, const uint16_t *__restrict__ X, int B,
                                        int Bp, int n_active, int D, int64_t Mp, float scale, float *__restrict__ dW,
                                        const DwUpdate &up, const DwCells &cells) {
    const int tiles_n = (D + T::BN - 1) / T::BN;
    const int n_tiles = tiles_n * ((n_active + T::BM - 1) / T::BM);
    if (bid >= n_tiles) return;
    const int t = ks_xcd_remap(bid, n_tiles);
    const int tn = t % tiles_n, tm = t / tiles_n;
    // the classes of the tile's rows, for the update: requested before the first k-tile, straight into LDS behind the stages
    static_assert(T::NT == TileDw::NT && T::LDS_ELEMS + 2 * (T::BM + DW_CELL_SLOTS * 128) <= DW_LDS_ELEMS, "one launch shape for all tiles");
    int32_t *s_cls = (int32_t *)(lds + T::LDS_ELEMS);
    if (up.Wm && threadIdx.x < T::BM) {
        const int a = tm * T::BM + (int)threadIdx.x;
        __builtin_amdgcn_global_load_lds(KS_GPTR(up.idx + (a < n_active ? a : n_active - 1)),
                                         KS_LPTR(s_cls + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u)), 4, 0, 0);
    }
    KsAM8<T::BM, T::NW> ar;
    KsAKmaj<T::BN, T::NW> br;
    ar.init(dZ8, Bp, tm * T::BM, (int)Mp);
    br.init(X, D, nullptr, tn * T::BN, D, B, 0);
    f32x16_t acc[T::FM][T::FN];
    ks_a_clear<T>(acc);
    // Cells: lane l of a wavefront looks after sample l of the k-tile and the rows that the wavefront reads, so that its own
    // write before its own fragment reads is all the order it takes (wavefronts that share the rows write the same value).
    // The k-tiles' cells are requested two k-tiles ahead, by one wavefront each, and looked at one ahead.
    int32_t *const s_cells = s_cls + T::BM; // [slot][pos, val][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nk = (B + 63) / 64;
    const int m_first = tm * T::BM + wave / T::WAVES_N * T::WM; // the wavefront's first row
    auto cells_request = [&](int kt) __attribute__((always_inline)) {
        if (wave < 2 && kt < nk)
            __builtin_amdgcn_global_load_lds(KS_GPTR((wave ? (const int32_t *)cells.val : cells.pos) + kt * 64 + lane),
                                             KS_LPTR(s_cells + ((kt & (DW_CELL_SLOTS - 1)) * 2 + wave) * 64), 4, 0, 0);
    };
    int pos_next = -1; // of the lane's sample in the next k-tile; as read (a wait for it would stand here otherwise)
    auto place = [&](int kt, uint16_t *st) __attribute__((always_inline)) {
        const int32_t *const here = s_cells + (kt & (DW_CELL_SLOTS - 1)) * 128 + lane;
        const int pos = (kt == 0 ? here[0] : pos_next) - m_first;
        pos_next = s_cells[((kt + 1) & (DW_CELL_SLOTS - 1)) * 128 + lane]; // (beyond the last k-tile: not used)
        if ((unsigned)pos < (unsigned)T::WM && kt * 64 + lane < B) {
            const int m = wave / T::WAVES_N * T::WM + pos;
            // (as assembly, like the reads that must come after it)
            asm volatile("ds_write_b16 %0, %1" ::"v"(ks_lds_addr(st + (m >> 3) * KS_M8_SLAB + lane * 8 + (m & 7))), "v"(here[64]) : "memory");
        }
        cells_request(kt + 2);
    };
    // (samples B .. of the last k-tile: zeros of dZ8 meet the last row of X)
    if constexpr (CELLS) {
        cells_request(0);
        cells_request(1);
        ks_a_mainloop_il<T, KS_M8, KS_KMAJ, 2>(ar, br, 0, nk, lds, acc, place);
    } else {
        ks_a_mainloop_il<T, KS_M8, KS_KMAJ, 2>(ar, br, 0, nk, lds, acc);
    }
    // epilogue, row-wise through LDS: gradient rows out (if wanted) and, if asked for, the update of the master
    // rows and of their 16-bit copy.  Up to four rows per thread are in flight at a time, the next ones requested before
    // the present ones are stored (and the first before the slab is staged): 192 x 256 tiles of 17,425 rows 43 -> 40 us,
    // 256 x 256 of 124,580 rows 420 -> 350.  (Two at a time beside the 128 accumulators of a 256 x 256 tile: four spill.)
    typedef KsASlab<T> SL;
    float *st = (float *)lds;
    const int d_base = tn * T::BN;
    constexpr int PER = SL::ROWS * SL::QUADS / T::NT; // pieces per thread and slab
    constexpr int U = T::BM * T::BN > 192 * 256 ? 2 : (PER < 4 ? PER : 4), NB = PER / U; // batches per slab
    static_assert(SL::ROWS * SL::QUADS % T::NT == 0 && PER % U == 0, "slab shape");
    float4 wn[U];
    int cn[U]; // the classes of the next batch's pieces (-1: no piece)
    auto request = [&](int b) __attribute__((always_inline)) { // batch b of all slabs
        const int p = b / NB, q0 = b % NB * U;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = (q0 + u) * T::NT + threadIdx.x;
            const int row = p * SL::ROWS + q / SL::QUADS, d = d_base + q % SL::QUADS * 4;
            cn[u] = -1;
            if (tm * T::BM + row < n_active && d < D) cn[u] = up.Wm ? s_cls[row] : 0; // D % 4 == 0
            if (up.Wm) wn[u] = cn[u] >= 0 ? *(const float4 *)(up.Wm + (int64_t)cn[u] * D + d) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    request(0);
    for (int p = 0; p < T::WAVES_M; ++p) {
        ks_a_stage_slab<T>(acc, st, p);
        __syncthreads();
        for (int q0 = 0; q0 < PER; q0 += U) {
            float4 g[U], w[U];
            int cls[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                w[u] = wn[u];
                cls[u] = cn[u];
            }
            const int b = p * NB + q0 / U + 1;
            if (b < T::WAVES_M * NB) request(b);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = (q0 + u) * T::NT + threadIdx.x;
                const float4 v = ks_a_slab_quad<T>(st, q / SL::QUADS, q % SL::QUADS);
                g[u] = make_float4(scale * v.x, scale * v.y, scale * v.z, scale * v.w);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (cls[u] < 0) continue;
                const int q = (q0 + u) * T::NT + threadIdx.x, d = d_base + q % SL::QUADS * 4;
                if (dW) *(float4 *)(dW + (int64_t)(tm * T::BM + p * SL::ROWS + q / SL::QUADS) * D + d) = g[u];
                if (up.Wm) {
                    w[u].x = fmaf(up.alpha, g[u].x, w[u].x);
                    w[u].y = fmaf(up.alpha, g[u].y, w[u].y);
                    w[u].z = fmaf(up.alpha, g[u].z, w[u].z);
                    w[u].w = fmaf(up.alpha, g[u].w, w[u].w);
                    const int64_t at = (int64_t)cls[u] * D + d;
                    *(float4 *)(up.Wm + at) = w[u];
                    if (up.Wb) *(uint2 *)(up.Wb + at) = make_uint2(ks_pack_bf2(w[u].x, w[u].y), ks_pack_bf2(w[u].z, w[u].w));
                }
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------
// stand-alone row gather (Algorithm 1's W_active as a dense matrix); one wavefront per row
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(SM_NT)
gather_rows_kernel(const uint16_t *__restrict__ W, const int32_t *__restrict__ active_idx,
                   const int32_t *__restrict__ n_active_p, int M, int64_t C, int D, uint16_t *__restrict__ out,
                   int32_t *dev_status) {
    const int n = sm_clamp_n(n_active_p, M);
    const int a = blockIdx.x * (SM_NT / 64) + (threadIdx.x >> 6);
    if (a >= n) return;
    const int32_t c = active_idx[a];
    if (c < 0 || c >= C) {
        if ((threadIdx.x & 63) == 0) ks_flag(dev_status, KS_DEV_BAD_INDEX);
        return;
    }
    const uint4 *src = (const uint4 *)(W + (int64_t)c * D);
    uint4 *dst = (uint4 *)(out + (int64_t)a * D);
    for (int q = threadIdx.x & 63; q < D / 8; q += 64) dst[q] = src[q];
}

// identity active list for the full-softmax entry point
__global__ void __launch_bounds__(SM_NT)
full_prepare_kernel(const int32_t *__restrict__ labels, int64_t C, int B, int32_t *active_idx, int32_t *n_active,
                    int32_t *target_pos, int32_t *dev_status) {
    int64_t t = (int64_t)blockIdx.x * SM_NT + threadIdx.x;
    if (t == 0) *n_active = (int32_t)C;
    if (t < C) active_idx[t] = (int32_t)t;
    if (t < B) {
        int32_t y = labels[t];
        if (y < 0 || y >= C) { ks_flag(dev_status, KS_DEV_BAD_LABEL); y = 0; }
        target_pos[t] = y;
    }
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
// two-sweep softmax, split over nodes: what goes out after the statistics sweep, what comes in before the
// gradient sweep.  (lse_i, 1) is a valid (max, sum) pair: sum_a exp(z_ia - lse_i) = 1.
__global__ void __launch_bounds__(SM_NT)
sm_export_kernel(const float *__restrict__ lse, const float *__restrict__ zt, const int32_t *__restrict__ target_pos,
                 const int32_t *__restrict__ n_active_p, int M, int B, SmSplitIO io) {
    const int i = blockIdx.x * SM_NT + threadIdx.x;
    if (i >= B) return;
    const int n = sm_clamp_n(n_active_p, M);
    const int tp = target_pos[i];
    io.row_max[i] = n > 0 ? lse[i] : -INFINITY;
    io.row_sum[i] = n > 0 ? 1.f : 0.f;
    io.tz_out[i] = (tp >= 0 && tp < n) ? zt[i] : 0.f;
}
__global__ void __launch_bounds__(SM_NT)
sm_import_kernel(SmSplitIO io, int B, float *__restrict__ lse, float *__restrict__ loss_i) {
    const int i = blockIdx.x * SM_NT + threadIdx.x;
    if (i >= B) return;
    const float l = io.gmax[i] + __logf(io.gsum[i]);
    lse[i] = l;
    loss_i[i] = l - io.gtz[i];
}
// caller-supplied selection: ids outside [0, C) and positions outside the list are flagged and made harmless
__global__ void __launch_bounds__(SM_NT)
sm_sanitize_kernel(const int32_t *__restrict__ active_idx, const int32_t *__restrict__ n_active_p,
                   const int32_t *__restrict__ target_pos, int64_t C, int M, int B, int32_t *__restrict__ act_safe,
                   int32_t *__restrict__ n_safe, int32_t *__restrict__ tp_safe, int32_t *dev_status) {
    const int t = blockIdx.x * SM_NT + threadIdx.x;
    // (all three loads are issued before the count is looked at: the kernel is one round trip to memory long)
    const int32_t a_in = t < M ? active_idx[t] : -1;
    const int32_t tp_in = t < B ? target_pos[t] : -1;
    int n = *n_active_p;
    if (n < 0 || n > M) {
        if (t == 0) ks_flag(dev_status, KS_DEV_BAD_COUNT);
        n = n < 0 ? 0 : M;
    }
    if (t == 0) *n_safe = n;
    if (t < M) {
        int32_t a = -1;
        if (t < n) {
            a = a_in;
            if (a < 0 || a >= C) {
                ks_flag(dev_status, KS_DEV_BAD_INDEX);
                a = 0;
            }
        }
        act_safe[t] = a;
    }
    if (t < B) {
        int32_t tp = tp_in;
        if (tp >= n) {
            ks_flag(dev_status, KS_DEV_BAD_LABEL);
            tp = -1;
        }
        tp_safe[t] = tp < 0 ? -1 : tp;
    }
}

// compute units of the current device (asked once)
static int ks_n_cu() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            n = v;
        else
            n = 256;
    }
    return n;
}

// Whether the softmax runs as sweeps with resident samples: a sample block's fragments fit in registers up to D = 512, every
// block of 256 samples needs a workgroup, and the sweeps take logarithms of the two factors.  (NaN factors: no.)
static bool sm_sweeps(int D, int B, float scale, float grad_scale) {
    return D <= 512 && ks_ceil_div(B, 256) <= SM_SOE_GRID && scale > 0.f && grad_scale / (float)B > 0.f;
}
// The fast path: those sweeps, or else the tile engine, whose k-tiles are whole (D % 64 == 0).  What neither takes -- an odd
// multiple of 32 with grad_scale <= 0 (a loss without gradients, ascent), scale <= 0 or more than 65,536 samples, or beyond
// 512 -- is left to the generic path.
static bool sm_fast(int D, int B, float scale, float grad_scale) { return D % 64 == 0 || sm_sweeps(D, B, scale, grad_scale); }

struct SmWs {
    void *select;
    float *Z;
    uint16_t *dZ;
    float *lse;
    float *part;
    uint16_t *dZ8; // fast path: the logit gradient is kept transposed only
    float *pm, *pl, *zt; // fast path: per class-tile softmax statistics, target logits
    float *inv;          // one-sweep softmax: 1 / sum_a exp(z_ia - scale) per sample
    uint16_t *X2;        // one-sweep softmax: rows of X scaled by that
    float *kept;         // two-sweep softmax of a small problem: the first sweep's products
    int32_t *cell_pos;   // one-sweep softmax: the target entries (DwCells)
    uint32_t *cell;
    int S;
    int64_t Mp;
    int Bp;
    bool fast;
    size_t bytes;
};

// dX tiles of 256 x 256 instead of 128 x 128.  The contraction is bound by the load requests of its operands: a wide tile has
// half of them per flop, and its share of the active rows is twice as long, so half the partial products travel.  One workgroup
// per compute unit, so 16 tiles (B = 2,048 at D = 512) are needed for 16 shares to fill the chip; fewer tiles mean more shares,
// whose partial products cost what the loads save.  So do short lists (narrow tiles have fewer shares then).  Whole steps at
// D = 512, narrow -> wide: B = 2,048, M = 32,768: 302 -> 305 us (stays narrow); B = 1,793, M = 60,000: 460 -> 427; B = 4,000,
// M = 50,001: 1,041 -> 905; B = 2,048, M = 131,072: 1,081 -> 971; D = 256, B = 4,000, M = 65,536: 617 -> 592.
static bool sm_dx_wide(int B, int D, int64_t M) {
    return D % 256 == 0 && ks_ceil_div(B, TileDxWide::BM) * (D / TileDxWide::BN) >= 16 && M >= 49152;
}

static int sm_splits(int B, int D, int64_t M, bool fast) {
    if (fast && sm_dx_wide(B, D, M)) {
        const int tiles = (int)ks_ceil_div(B, TileDxWide::BM) * (D / TileDxWide::BN);
        const int S = (int)ks_ceil_div(256, tiles), need = (int)ks_ceil_div(ks_ceil_div(M, 64), DxIdx<TileDxWide>::CAP / 64);
        return S > need ? S : need;
    }
    int tiles = fast ? (int)(ks_ceil_div(B, TileDx::BM) * ks_ceil_div(D, TileDx::BN))
                     : (int)(ks_ceil_div(B, TileG::BM) * ks_ceil_div(D, TileG::BN));
    // two workgroups per compute unit
    int S = (int)ks_ceil_div(512, tiles);
    if (S < 1) S = 1;
    if (S > 32) S = 32;
    if (fast) { // a share of the active dimension must fit the dX kernel's LDS index cache
        const int64_t nk = ks_ceil_div(M, 64);
        const int need = (int)ks_ceil_div(nk, DxIdx<TileDx>::CAP / 64);
        if (S < need) S = need;
    }
    return S;
}

// Whether the two-sweep softmax keeps its products instead of forming them again.  It spares a launch (the merge, 4 us) and the
// second sweep's set-up, and costs 10 bytes of traffic per product against 2 D operations: it pays up to a million products or
// 32 D^2, whichever is more.  Whole calls, us, sweep -> kept, inside: 900 classes x 64, batch 256: 26.7 -> 23.3; 4,096 x 64, 256:
// 28.5 -> 26.4; 2,000 x 128, 512: 33.3 -> 30.6; 8,192 x 256, 180: 38.1 -> 37.1; 3,000 x 320, 400: 43.9 -> 37.8; 16,384 x 384, 256: 55.8 ->
// 56.0; 4,096 x 512, 128: 41.8 -> 34.6; 24,000 x 512, 256: 74.3 -> 73.0; 16,384 x 512, 512: 82.6 -> 76.0; beyond: 4,096 x 64, 512: 31.3 ->
// 32.1; 8,192 x 128, 256: 32.1 -> 34.5; 12,000 x 256, 512: 46.0 -> 48.3; 24,000 x 320, 256: 61.5 -> 64.1; 24,000 x 384, 256: 64.3 -> 66.3;
// 32,319 x 512, 1,024: 212 -> 216.  (By the cap M: the active count is known to the device only, and with fewer both get faster.)
// Bytes of the array (0: not kept), at most 34 MB.
static size_t sm_kept_bytes(int B, int D, int64_t M) {
    const int64_t n = (int64_t)ks_align_up((size_t)B, KS_BP_ALIGN) * sm_mp(M);
    return D <= 512 && (n <= 1 << 20 || n <= 32 * (int64_t)D * D) ? (size_t)n * sizeof(float) : 0;
}

static SmWs sm_carve(void *ws, int64_t C, int D, int B, int K, int64_t M, bool with_select, bool fast) {
    KsArena ar(ws);
    SmWs w;
    w.fast = fast;
    w.Mp = sm_mp(M);
    w.Bp = (int)ks_align_up((size_t)B, KS_BP_ALIGN);
    w.S = sm_splits(B, D, M, w.fast);
    w.select = with_select ? (void *)ar.take<char>(ks_select_ws_bytes(C, B, K)) : nullptr;
    w.lse = ar.take<float>((size_t)B);
    w.part = ar.take<float>((size_t)(w.S + (fast ? 1 : 0)) * B * D); // (the one-sweep softmax adds a product: SmCombine)
    w.Z = nullptr;
    w.dZ = w.dZ8 = nullptr;
    w.pm = w.pl = w.zt = w.inv = nullptr;
    w.X2 = nullptr;
    w.kept = nullptr; // see sm_take_kept
    w.cell_pos = nullptr;
    w.cell = nullptr;
    if (w.fast) {
        w.dZ8 = ar.take<uint16_t>((size_t)w.Mp * w.Bp);
        size_t nt = (size_t)(w.Mp / TileSm::BM);
        if (nt < (size_t)SM_SOE_GRID) nt = SM_SOE_GRID; // per-slab statistics of the stationary-operand kernels
        w.pm = ar.take<float>(nt * w.Bp);
        w.pl = ar.take<float>(nt * w.Bp);
        w.zt = ar.take<float>((size_t)w.Bp);
        w.inv = ar.take<float>((size_t)w.Bp);
        w.X2 = ar.take<uint16_t>((size_t)w.Bp * D);
        w.cell_pos = ar.take<int32_t>((size_t)w.Bp);
        w.cell = ar.take<uint32_t>((size_t)w.Bp);
    } else {
        w.Z = ar.take<float>((size_t)B * w.Mp);
        w.dZ = ar.take<uint16_t>((size_t)B * w.Mp);
    }
    w.bytes = ar.off;
    return w;
}
// bytes of the workspace: the factors, which decide between the paths of an odd multiple of 32, are not known to the callers'
// size queries, so it holds either
static size_t sm_bytes(int64_t C, int D, int B, int K, int64_t M, bool with_select) {
    const size_t fast = D <= 512 || D % 64 == 0 ? sm_carve(nullptr, C, D, B, K, M, with_select, true).bytes : 0;
    const size_t generic = D % 64 != 0 ? sm_carve(nullptr, C, D, B, K, M, with_select, false).bytes : 0;
    return fast > generic ? fast : generic;
}
// The kept products lie behind everything else, and only the size queries of the calls that can use them ask for their room:
// `need` bytes are enough to run, without the array the call sweeps twice.  (A workspace sized for a large batch serves a
// smaller one as well: the larger problem keeps nothing and may need less than the smaller one with its products.)
static size_t sm_with_kept(size_t need, int B, int D, int64_t M) {
    const size_t bytes = sm_kept_bytes(B, D, M);
    return bytes ? ks_align_up(need, 256) + bytes : need;
}
static void sm_take_kept(SmWs &w, void *ws, size_t need, size_t ws_bytes, int B, int D, int64_t M) {
    if (w.fast && sm_kept_bytes(B, D, M) && ws_bytes >= sm_with_kept(need, B, D, M)) w.kept = (float *)((char *)ws + ks_align_up(need, 256));
}

// Sweeps of a depth of up to eight k-tiles (D <= 512, D % 32 == 0): F(CFG) is instantiated for the depth's stage shape
#define SM_COMMA ,
#define SM_FOR_DEPTH(F)                                                                                   \
    do {                                                                                                  \
        const int kt = (D + 63) / 64;                                                                     \
        if (D % 64 == 0) {                                                                                \
            if (kt == 1) F(SmSoe<1 SM_COMMA false>); else if (kt == 2) F(SmSoe<2 SM_COMMA false>);        \
            else if (kt == 3) F(SmSoe<3 SM_COMMA false>); else if (kt == 4) F(SmSoe<4 SM_COMMA false>);   \
            else if (kt == 5) F(SmSoe<5 SM_COMMA false>); else if (kt == 6) F(SmSoe<6 SM_COMMA false>);   \
            else if (kt == 7) F(SmSoe<7 SM_COMMA false>); else F(SmSoe<8 SM_COMMA false>);                \
        } else {                                                                                          \
            if (kt == 1) F(SmSoe<1 SM_COMMA true>); else if (kt == 2) F(SmSoe<2 SM_COMMA true>);          \
            else if (kt == 3) F(SmSoe<3 SM_COMMA true>); else if (kt == 4) F(SmSoe<4 SM_COMMA true>);     \
            else if (kt == 5) F(SmSoe<5 SM_COMMA true>); else if (kt == 6) F(SmSoe<6 SM_COMMA true>);     \
            else if (kt == 7) F(SmSoe<7 SM_COMMA true>); else F(SmSoe<8 SM_COMMA true>);                  \
        }                                                                                                 \
    } while (0)

// everything after the selection; active_idx / n_active / target_pos are device-resident inputs here
static int sm_run(const uint16_t *W, const uint16_t *X, int D, int B, int64_t M, float scale, float grad_scale,
                  const int32_t *active_idx, const int32_t *n_active, const int32_t *target_pos,
                  float *loss_per_sample, float *loss_mean, float *dX, float *dW_active, const SmWs &w,
                  uint32_t flags, int32_t *dev_status, hipStream_t st, hipEvent_t *ev = nullptr, int mode = SM_WHOLE,
                  SmSplitIO io = SmSplitIO(), DwUpdate up = DwUpdate(), const KsSelNext *next_p = nullptr) {
    auto mark = [&](int k) { if (ev) (void)hipEventRecord(ev[k], st); };
    KsSelNext next = KsSelNext();
    if (next_p) next = *next_p; // (the caller has checked that this path takes it: w.fast, and the dX and dW launches are made)
    if (mode != SM_WHOLE && !w.fast) return KS_UNSUPPORTED;
    if (mode == SM_EXPORT) loss_per_sample = w.inv; // not known before the exchange: the kernels' loss output is scratch
    const int Mi = (int)M;
    const float g = grad_scale / (float)B;
    bool fused = false;
    SmCombine comb = SmCombine();
    int S = w.S; // shares of the active classes in dX
    if (w.fast) {
        const int tiles_s = (int)ks_ceil_div(B, 256);
        const bool soe = sm_sweeps(D, B, scale, grad_scale);
        // One sweep: unit rows (|logit| <= scale, and exp(-2 scale) must stay a normal number) of 128, 256 or 512.  It rounds more
        // than two sweeps do: X / sum becomes a bf16 operand of dW, and the own class's gradient is minus the sum of the others
        // in bf16 (dX and dW 2 to 3 parts in 1,000 from the two-sweep results, which are 1 in 10,000 from exact ones).  Callers at
        // those depths have chosen that with the flag; at the other ones the flag has no effect.
        fused = soe && (D == 128 || D == 256 || D == 512) && (flags & KS_FLAG_UNIT_ROWS) && scale <= KS_FUSED_MAX_SCALE;
        const int grid = soe ? SM_SOE_GRID / tiles_s * tiles_s : 0, slabs = soe ? grid / tiles_s : 0;
        if (fused) {
#define SM_FUSED_LAUNCH(CFG)                                                                                              \
    hipLaunchKernelGGL((sm_fused_soe_kernel<CFG>), dim3(grid), dim3(512), 0, st, X, W, active_idx, n_active, target_pos, B, \
                       w.Bp, D, Mi, tiles_s, scale, w.pl, w.pm, w.dZ8)
            if (mode != SM_IMPORT) { // the first call of a split has left the exponentials in the workspace
                if (D == 512) SM_FUSED_LAUNCH(SmSoe<8 SM_COMMA false>);
                else if (D == 256) SM_FUSED_LAUNCH(SmSoe<4 SM_COMMA false>);
                else SM_FUSED_LAUNCH(SmSoe<2 SM_COMMA false>);
            }
#undef SM_FUSED_LAUNCH
            mark(2);
            comb.pl = w.pl;
            comb.pl_others = w.pm;
            comb.slabs = slabs;
            comb.D = D;
            comb.target_pos = target_pos;
            comb.X = X;
            comb.scale = scale;
            comb.inv_sum = w.inv;
            comb.loss_i = loss_per_sample;
            comb.X2 = w.X2;
            comb.cell_pos = w.cell_pos;
            comb.cell = w.cell;
            comb.dev_status = dev_status;
            comb.mode = mode;
            comb.io = io;
            // Narrow dX tiles are two to a compute unit.  Where the tiles and workgroups of few samples are more than that, and
            // workgroups of many samples fit beside them, with a twelfth less shares for the tiles if that does it, all run at once.
            // Where they do not, or where the shares are short, the long chain of many samples only delays the launch's end.
            // Whole calls, us, few -> many: D = 512, B = 1,024: A = 2,000: 44.4 -> 46.4; 9,000: 69.6 -> 69.3; 17,425: 97.5 -> 96.2 (15
            // shares instead of 16); D = 512, B = 512: 2,000: 39.8 -> 42.6; 17,425: 69.4 -> 68.4 (31 for 32); D = 256, B = 777: 2,000:
            // 37.1 -> 39.2; 4,737: 40.2 -> 39.8; 17,425: 65.5 -> 63.6; D = 128, B = 1,536: 4,737: 48.3 -> 46.9; and where they do not fit:
            // D = 512, B = 2,048: 4,737: 77.4 -> 84.0; 17,425: 153.9 -> 156.5; D = 256, B = 2,048: 9,000: 75.0 -> 77.8; D = 512, B = 777:
            // 17,425: 95.6 -> 97.2; B = 1,536: 139.6 -> 141.3.
            const bool wide = sm_dx_wide(B, D, M);
            const int tiles = (int)(ks_ceil_div(B, TileDx::BM) * ks_ceil_div(D, TileDx::BN)), slots = 2 * 256;
            const int few = (int)ks_ceil_div(B, SM_CF_FEW), many = (int)ks_ceil_div(B, SM_CF_MANY);
            const int room = tiles * S <= slots ? (slots - many) / tiles : 0, fit = room < S ? room : S; // shares that leave room
            comb.many = mode != SM_EXPORT && (wide || (tiles * S + few > slots && fit > 0 && fit >= S - S / 12 && M >= 128 * (int64_t)S &&
                                                       (int64_t)fit * DxIdx<TileDx>::CAP >= M));
            comb.blocks = comb.many ? many : few;
            if (!wide && comb.many) S = fit;
            comb.extra = w.part + (int64_t)S * B * D;
            if (mode == SM_EXPORT) {
                hipLaunchKernelGGL(sm_combine_fused_kernel, dim3((unsigned)comb.blocks), dim3(SM_CF_NT), 0, st, comb, n_active, Mi, B,
                                   w.Bp, active_idx, W);
                mark(3);
                KS_LAUNCH_CHECK();
                return KS_OK;
            }
            mark(3);
        } else if (soe) {
            const bool keep = mode == SM_WHOLE && w.kept;
            if (mode != SM_IMPORT) {
#define SM_STATS_LAUNCH(CFG)                                                                                              \
    do {                                                                                                                  \
        if (keep)                                                                                                         \
            hipLaunchKernelGGL((sm_stats_soe_kernel<CFG, true>), dim3(grid), dim3(512), 0, st, X, W, active_idx, n_active, target_pos, \
                               B, w.Bp, D, Mi, tiles_s, scale, w.pm, w.pl, w.zt, w.kept);                                 \
        else                                                                                                              \
            hipLaunchKernelGGL((sm_stats_soe_kernel<CFG, false>), dim3(grid), dim3(512), 0, st, X, W, active_idx, n_active, target_pos, \
                               B, w.Bp, D, Mi, tiles_s, scale, w.pm, w.pl, w.zt, w.kept);                                 \
    } while (0)
                SM_FOR_DEPTH(SM_STATS_LAUNCH);
#undef SM_STATS_LAUNCH
                mark(2);
                if (!keep)
                    hipLaunchKernelGGL(sm_combine_soe_kernel, dim3((unsigned)ks_ceil_div(B, SM_NT / 64)), dim3(SM_NT), 0, st,
                                       w.pm, w.pl, w.zt, n_active, Mi, slabs, B, w.Bp, w.lse, loss_per_sample);
                mark(3);
            } else {
                hipLaunchKernelGGL(sm_import_kernel, dim3((unsigned)ks_ceil_div(B, SM_NT)), dim3(SM_NT), 0, st, io, B, w.lse,
                                   loss_per_sample);
            }
            if (keep) {
                const int sbs = (B + 63) / 64 * 2, groups = (int)ks_ceil_div(M, 128); // class blocks in fours
                const int gy = (int)ks_ceil_div(1024, sbs);
                hipLaunchKernelGGL(sm_grad_kept_kernel, dim3(sbs, gy < groups ? gy : groups), dim3(SM_NT), 0, st, w.kept, w.pm, w.pl,
                                   w.zt, n_active, target_pos, B, w.Bp, Mi, slabs, scale, g, loss_per_sample, w.dZ8);
            } else if (mode != SM_EXPORT) {
#define SM_GRAD_LAUNCH(CFG)                                                                                               \
    hipLaunchKernelGGL((sm_grad_soe_kernel<CFG>), dim3(grid), dim3(512), 0, st, X, W, active_idx, n_active, target_pos,     \
                       w.lse, B, w.Bp, D, Mi, tiles_s, scale, g, w.dZ8)
                SM_FOR_DEPTH(SM_GRAD_LAUNCH);
#undef SM_GRAD_LAUNCH
            }
        } else {
            typedef TileSm T;
            const int tiles = (int)(ks_ceil_div(B, T::BN) * ks_ceil_div(M, T::BM));
            if (mode != SM_IMPORT) {
                hipLaunchKernelGGL(sm_stats_kernel<T>, dim3(tiles), dim3(T::NT), 0, st, X, W, active_idx, n_active, target_pos,
                                   B, w.Bp, D, Mi, scale, w.pm, w.pl, w.zt);
                mark(2);
                hipLaunchKernelGGL(sm_combine_kernel, dim3((unsigned)ks_ceil_div(B, SM_NT / 64)), dim3(SM_NT), 0, st, w.pm,
                                   w.pl, w.zt, n_active, Mi, T::BM, B, w.Bp, w.lse, loss_per_sample);
                mark(3);
            } else {
                hipLaunchKernelGGL(sm_import_kernel, dim3((unsigned)ks_ceil_div(B, SM_NT)), dim3(SM_NT), 0, st, io, B, w.lse,
                                   loss_per_sample);
            }
            if (mode != SM_EXPORT)
                hipLaunchKernelGGL(sm_grad_kernel<T>, dim3(tiles), dim3(T::NT), 0, st, X, W, active_idx, n_active, target_pos,
                                   w.lse, B, w.Bp, D, Mi, scale, g, w.dZ8);
        }
        if (mode == SM_EXPORT) { // two-sweep paths: the statistics sweep is done, (lse, 1) and the target logit go out
            hipLaunchKernelGGL(sm_export_kernel, dim3((unsigned)ks_ceil_div(B, SM_NT)), dim3(SM_NT), 0, st, w.lse, w.zt,
                               target_pos, n_active, Mi, B, io);
            KS_LAUNCH_CHECK();
            return KS_OK;
        }
        mark(4);
        {
            auto dx = [&](auto tile) {
                typedef decltype(tile) T;
                const int tiles = (int)(ks_ceil_div(B, T::BM) * ks_ceil_div(D, T::BN));
                if (next.nsel) next.nfetch = (int)ks_ceil_div((int64_t)next.B * (next.K + 1), (int64_t)T::NT);
                hipLaunchKernelGGL(dx_partial_async_kernel<T>, dim3(comb.blocks + tiles * S + next.nfetch), dim3(T::NT), 0, st, w.dZ8,
                                   w.Bp, W, active_idx, n_active, B, D, Mi, S, w.part, comb, next);
            };
            if (sm_dx_wide(B, D, M)) dx(TileDxWide());
            else dx(TileDx());
        }
        mark(5);
        mark(6); // the reduction of the partial products rides along with the next launch
        {
            typedef TileDw T;
            // workgroups for 128-row tiles, or, where those leave compute units without one, for as many tiles of the smallest shape
            int tiles = (int)(ks_ceil_div(M, TileDw128::BM) * ks_ceil_div(D, T::BN));
            const int least = (int)(ks_ceil_div(M, TileDw64n::BM) * ks_ceil_div(D, TileDw64n::BN)), n_cu = ks_n_cu();
            if (tiles < n_cu) tiles = least < n_cu ? least : n_cu;
            DxReduceJob job;
            job.part = w.part;
            job.S = S + (fused ? 1 : 0);
            job.BD = (int64_t)B * D;
            job.scale = fused ? scale * g : scale;
            job.row_factor = fused ? w.inv : nullptr;
            job.dX = dX;
            job.loss_i = loss_per_sample;
            job.loss_mean = loss_mean;
            const dim3 grid(next.nsel + tiles + DW_REDUCE_BLOCKS);
            if (fused)
                hipLaunchKernelGGL(dw_async_kernel<true>, grid, dim3(T::NT), 0, st, w.dZ8, w.X2, B, w.Bp, n_active, D, Mi, w.Mp,
                                   scale * g, dW_active, tiles, n_cu, job, up, DwCells{w.cell_pos, w.cell}, next);
            else
                hipLaunchKernelGGL(dw_async_kernel<false>, grid, dim3(T::NT), 0, st, w.dZ8, X, B, w.Bp, n_active, D, Mi, w.Mp, scale,
                                   dW_active, tiles, n_cu, job, up, DwCells(), next);
        }
        mark(7);
        KS_LAUNCH_CHECK();
        return KS_OK;
    }
    typedef TileG T;
    const int tiles_b = (int)ks_ceil_div(B, T::BM);
    const int tiles_a_n = (int)ks_ceil_div(M, T::BN), tiles_a_m = (int)ks_ceil_div(M, T::BM);
    const int tiles_d = (int)ks_ceil_div(D, T::BN);

    hipLaunchKernelGGL(logits_kernel<T>, dim3(tiles_b * tiles_a_n), dim3(T::NT), 0, st, X, W, active_idx, n_active, B, D,
                       Mi, scale, w.Z, w.Mp);
    mark(2);
    hipLaunchKernelGGL(row_stats_kernel, dim3(B), dim3(SM_NT), 0, st, w.Z, w.Mp, n_active, Mi, target_pos, w.lse,
                       loss_per_sample);
    mark(3);
    hipLaunchKernelGGL(dz_kernel, dim3((unsigned)ks_ceil_div(w.Mp, SM_NT * 8), B < 65535 ? B : 65535), dim3(SM_NT), 0, st, w.Z, w.Mp,
                       n_active, B, Mi, target_pos, w.lse, g, w.dZ);
    mark(4);
    hipLaunchKernelGGL(dx_partial_kernel<T>, dim3(tiles_b * tiles_d, w.S), dim3(T::NT), 0, st, w.dZ, w.Mp, W, active_idx,
                       n_active, B, D, Mi, w.part);
    mark(5);
    hipLaunchKernelGGL(dx_reduce_kernel, dim3((unsigned)ks_ceil_div((int64_t)B * D / 4, SM_NT)), dim3(SM_NT), 0, st, w.part,
                       w.S, (int64_t)B * D, scale, (const float *)nullptr, D, dX, loss_per_sample, B, loss_mean);
    mark(6);
    hipLaunchKernelGGL(dw_kernel<T>, dim3(tiles_a_m * tiles_d), dim3(T::NT), 0, st, w.dZ, w.Mp, X, n_active, B, D, Mi,
                       scale, dW_active);
    mark(7);
    KS_LAUNCH_CHECK();
    return KS_OK;
}

static int sm_check_dims(int64_t C, int D, int B) {
    if (C < 1 || C >= (int64_t)1 << 31 || D < 32 || D % 32 != 0 || B < 1) return KS_INVALID_ARG;
    return KS_OK;
}

extern "C" size_t knn_softmax_workspace(int64_t C, int D, int B, int K, int M) {
    if (sm_check_dims(C, D, B) != KS_OK || K < 0 || M < 1) return 0;
    return sm_with_kept(sm_bytes(C, D, B, K, M, true), B, D, M);
}

static int sm_fwd_bwd(const uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *labels, const int32_t *graph,
                      int64_t C, int D, int B, int K, int M, float scale, float grad_scale, uint32_t flags,
                      int32_t *active_idx, int32_t *n_active, int32_t *target_pos, float *loss_per_sample,
                      float *loss_mean, float *dX, float *dW_active, void *ws, size_t ws_bytes, int32_t *dev_status,
                      void *stream, hipEvent_t *ev, float *W_master = nullptr, uint16_t *W_bf16_out = nullptr,
                      float alpha = 0.f) {
    if (!W_bf16 || !X_bf16 || !labels || !active_idx || !n_active || !target_pos || !loss_per_sample || !loss_mean ||
        !dX || !ws)
        return KS_INVALID_ARG;
    if (!dW_active && !(W_master && D % 64 == 0)) return KS_INVALID_ARG;
    if (sm_check_dims(C, D, B) != KS_OK || K < 0 || M < 1) return KS_INVALID_ARG;
    if (K > 0 && !graph) return KS_INVALID_ARG;
    if (B > M || (int64_t)K + 1 > M) return KS_INVALID_ARG;
    const size_t need = sm_bytes(C, D, B, K, M, true);
    if (ws_bytes < need) return KS_WORKSPACE_TOO_SMALL;
    const bool fast = sm_fast(D, B, scale, grad_scale); // the update runs inside the dW kernel of this path
    SmWs w = sm_carve(ws, C, D, B, K, M, true, fast);
    sm_take_kept(w, ws, need, ws_bytes, B, D, M);
    hipStream_t st = (hipStream_t)stream;
    if (ev) (void)hipEventRecord(ev[0], st);
    int rc = ks_select_launch(labels, graph, C, B, K, M, active_idx, n_active, target_pos, w.select, dev_status, st);
    if (rc != KS_OK) return rc;
    if (ev) (void)hipEventRecord(ev[1], st);
    DwUpdate up = DwUpdate();
    if (W_master && fast) {
        up.Wm = W_master;
        up.Wb = W_bf16_out;
        up.idx = active_idx;
        up.alpha = alpha;
    }
    rc = sm_run(W_bf16, X_bf16, D, B, M, scale, grad_scale, active_idx, n_active, target_pos, loss_per_sample, loss_mean,
                dX, dW_active, w, flags, dev_status, st, ev, SM_WHOLE, SmSplitIO(), up);
    if (rc != KS_OK || !W_master || fast) return rc;
    // other shapes: the stand-alone update on the stored gradient (active_idx is strictly ascending)
    return apply_weight_grad(W_master, W_bf16_out, active_idx, n_active, M, dW_active, alpha, C, D, 1, ws, ws_bytes,
                             dev_status, stream);
}

extern "C" int knn_softmax_fwd_bwd(const uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *labels,
                                   const int32_t *graph, int64_t C, int D, int B, int K, int M, float scale,
                                   float grad_scale, uint32_t flags, int32_t *active_idx, int32_t *n_active,
                                   int32_t *target_pos, float *loss_per_sample, float *loss_mean, float *dX,
                                   float *dW_active, void *ws, size_t ws_bytes, int32_t *dev_status, void *stream) {
    return sm_fwd_bwd(W_bf16, X_bf16, labels, graph, C, D, B, K, M, scale, grad_scale, flags, active_idx, n_active,
                      target_pos, loss_per_sample, loss_mean, dX, dW_active, ws, ws_bytes, dev_status, stream, nullptr);
}

extern "C" int knn_softmax_fwd_bwd_update(float *W_master, uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *labels,
                                          const int32_t *graph, int64_t C, int D, int B, int K, int M, float scale,
                                          float grad_scale, float alpha, uint32_t flags, int32_t *active_idx,
                                          int32_t *n_active, int32_t *target_pos, float *loss_per_sample, float *loss_mean,
                                          float *dX, float *dW_active, void *ws, size_t ws_bytes, int32_t *dev_status,
                                          void *stream) {
    if (!W_master) return KS_INVALID_ARG;
    return sm_fwd_bwd(W_bf16, X_bf16, labels, graph, C, D, B, K, M, scale, grad_scale, flags, active_idx, n_active,
                      target_pos, loss_per_sample, loss_mean, dX, dW_active, ws, ws_bytes, dev_status, stream, nullptr,
                      W_master, W_bf16, alpha);
}

extern "C" int knn_softmax_fwd_bwd_profiled(float *W_master, uint16_t *W_bf16, const uint16_t *X_bf16,
                                            const int32_t *labels, const int32_t *graph, int64_t C, int D, int B, int K,
                                            int M, float scale, float grad_scale, float alpha, uint32_t flags,
                                            int32_t *active_idx, int32_t *n_active, int32_t *target_pos,
                                            float *loss_per_sample, float *loss_mean, float *dX, float *dW_active, void *ws,
                                            size_t ws_bytes, int32_t *dev_status, void *stream, void **events,
                                            int n_events) {
    if (!events || n_events < KS_N_PHASE_EVENTS) return KS_INVALID_ARG;
    for (int k = 0; k < KS_N_PHASE_EVENTS; ++k)
        if (!events[k]) return KS_INVALID_ARG;
    return sm_fwd_bwd(W_bf16, X_bf16, labels, graph, C, D, B, K, M, scale, grad_scale, flags, active_idx, n_active,
                      target_pos, loss_per_sample, loss_mean, dX, dW_active, ws, ws_bytes, dev_status, stream,
                      (hipEvent_t *)events, W_master, W_bf16, alpha);
}

// whether the next batch's selection can run inside the step's launches: its bitmap fits a workgroup's LDS, its staged
// candidates the workspace
static bool sm_next_rides(int64_t C, int B, int K) {
    return sel1_fits(C, B) && ks_select_ws_bytes(C, B, K) >= (size_t)B * (K + 1) * sizeof(int32_t);
}
// The two calls of the softmax split over nodes.  Workspace: the softmax buffers (which carry the first call's
// exponentials, or nothing on the two-sweep paths, to the second call), then the sanitised copy of the selection.
struct SmSplitWs {
    SmWs w;
    int32_t *act, *n, *tp;
};
static SmSplitWs sm_split_carve(void *ws, int64_t C, int D, int B, int64_t M, bool fast, size_t *total) {
    const size_t used = sm_bytes(C, D, B, 0, M, false);
    SmSplitWs s;
    s.w = sm_carve(ws, C, D, B, 0, M, false, fast);
    KsArena ar(ws ? (void *)((char *)ws + used) : nullptr);
    s.act = ar.take<int32_t>((size_t)M);
    s.tp = ar.take<int32_t>((size_t)B);
    s.n = ar.take<int32_t>(1);
    if (total) *total = used + ar.off;
    return s;
}
static int sm_split_check(int64_t C, int D, int B, int M, float scale, uint32_t flags) {
    if (sm_check_dims(C, D, B) != KS_OK || M < 1 || !(scale > 0.f)) return KS_INVALID_ARG;
    if (flags & ~(uint32_t)KS_FLAG_UNIT_ROWS) return KS_INVALID_ARG;
    if (D % 64 != 0) return KS_UNSUPPORTED;
    return KS_OK;
}

extern "C" size_t knn_softmax_split_workspace(int64_t C, int D, int B, int M) {
    if (sm_split_check(C, D, B, M, 1.f, 0) != KS_OK) return 0;
    size_t total = 0;
    sm_split_carve(nullptr, C, D, B, M, true, &total);
    return total;
}

extern "C" int knn_softmax_fwd_stats(const uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *active_idx,
                                     const int32_t *n_active, const int32_t *target_pos, int64_t C, int D, int B, int M,
                                     float scale, uint32_t flags, float *row_max, float *row_sumexp, float *target_logit,
                                     void *ws, size_t ws_bytes, int32_t *dev_status, void *stream) {
    if (!W_bf16 || !X_bf16 || !active_idx || !n_active || !target_pos || !row_max || !row_sumexp || !target_logit || !ws)
        return KS_INVALID_ARG;
    const bool trusted = (flags & KS_FLAG_TRUSTED_LIST) != 0;
    flags &= ~(uint32_t)KS_FLAG_TRUSTED_LIST;
    int rc = sm_split_check(C, D, B, M, scale, flags);
    if (rc != KS_OK) return rc;
    size_t need = 0;
    SmSplitWs s = sm_split_carve(ws, C, D, B, M, true, &need);
    if (ws_bytes < need) return KS_WORKSPACE_TOO_SMALL;
    hipStream_t st = (hipStream_t)stream;
    const int nmax = M > B ? M : B;
    if (!trusted) {
        hipLaunchKernelGGL(sm_sanitize_kernel, dim3((unsigned)ks_ceil_div(nmax, SM_NT)), dim3(SM_NT), 0, st, active_idx,
                           n_active, target_pos, C, M, B, s.act, s.n, s.tp, dev_status);
        active_idx = s.act;
        n_active = s.n;
        target_pos = s.tp;
    }
    SmSplitIO io = SmSplitIO();
    io.row_max = row_max;
    io.row_sum = row_sumexp;
    io.tz_out = target_logit;
    return sm_run(W_bf16, X_bf16, D, B, M, scale, 1.f, active_idx, n_active, target_pos, nullptr, nullptr, nullptr, nullptr, s.w,
                  flags, dev_status, st, nullptr, SM_EXPORT, io);
}

// the next batch's selection on the node's compressed graph that rides along with the second call of a split (nullptr: none)
struct SmNextCsr {
    const int32_t *labels, *counts;
    const int64_t *offsets;
    const int32_t *flat;
    int64_t flat_len, Cg, c0;
    int K_max;
    uint32_t sel_flags;
    uint64_t pad_seed;
    int32_t *active_idx, *n_active, *n_found, *target_pos;
};
static int sm_bwd_from_stats(const uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *active_idx, const int32_t *n_active,
                             const int32_t *target_pos, const float *global_max, const float *global_sumexp,
                             const float *global_target_logit, int64_t C, int D, int B, int M, float scale, float grad_scale,
                             uint32_t flags, float *loss_per_sample, float *loss_mean, float *dX, float *dW_active,
                             const SmNextCsr *nx, void *ws, size_t ws_bytes, int32_t *dev_status, void *stream) {
    if (!W_bf16 || !X_bf16 || !active_idx || !n_active || !target_pos || !global_max || !global_sumexp ||
        !global_target_logit || !loss_per_sample || !loss_mean || !dX || !dW_active || !ws)
        return KS_INVALID_ARG;
    const bool trusted = (flags & KS_FLAG_TRUSTED_LIST) != 0;
    flags &= ~(uint32_t)KS_FLAG_TRUSTED_LIST;
    int rc = sm_split_check(C, D, B, M, scale, flags);
    if (rc != KS_OK) return rc;
    if (!(grad_scale > 0.f)) return KS_INVALID_ARG;
    if (nx) { // the conditions of knn_select_active_csr
        if (!nx->labels || !nx->counts || !nx->offsets || !nx->active_idx || !nx->n_active || !nx->target_pos) return KS_INVALID_ARG;
        if (nx->Cg < 1 || nx->Cg >= (int64_t)1 << 31 || nx->c0 < 0 || nx->c0 + C > nx->Cg) return KS_INVALID_ARG;
        if (nx->K_max < 0 || nx->flat_len < 0 || (nx->flat_len > 0 && !nx->flat)) return KS_INVALID_ARG;
        if (B > M || (int64_t)nx->K_max + 1 > M) return KS_INVALID_ARG;
        if (nx->sel_flags & ~(uint32_t)KS_FLAG_PAD_RANDOM) return KS_INVALID_ARG;
        if (trusted && (nx->active_idx == active_idx || nx->n_active == n_active || nx->target_pos == target_pos))
            return KS_INVALID_ARG; // a trusted list is read in place: the next one needs buffers of its own
    }
    size_t need = 0;
    SmSplitWs s = sm_split_carve(ws, C, D, B, M, true, &need);
    if (nx) need = ks_align_up(need, 256);
    void *sel_ws = (char *)ws + need;
    if (nx) need += ks_select_ws_bytes(C, B, nx->K_max);
    if (ws_bytes < need) return KS_WORKSPACE_TOO_SMALL;
    hipStream_t st = (hipStream_t)stream;
    const int nmax = M > B ? M : B;
    if (!trusted) {
        hipLaunchKernelGGL(sm_sanitize_kernel, dim3((unsigned)ks_ceil_div(nmax, SM_NT)), dim3(SM_NT), 0, st, active_idx,
                           n_active, target_pos, C, M, B, s.act, s.n, s.tp, dev_status);
        active_idx = s.act;
        n_active = s.n;
        target_pos = s.tp;
    }
    SmSplitIO io = SmSplitIO();
    io.gmax = global_max;
    io.gsum = global_sumexp;
    io.gtz = global_target_logit;
    KsSelNext next = KsSelNext();
    const bool ride = nx && sm_next_rides(C, B, nx->K_max);
    if (ride) {
        next.nsel = SEL1_GRID;
        next.csr_source = 1;
        next.csr = SelCsr{nx->labels, nx->counts, nx->offsets, nx->flat, nx->Cg, nx->c0, C, nx->flat_len, nx->K_max};
        next.pad = sel_pad_make((nx->sel_flags & KS_FLAG_PAD_RANDOM) != 0, C, nx->pad_seed);
        next.C = C;
        next.B = B;
        next.K = nx->K_max;
        next.M = M;
        next.cand = (int32_t *)sel_ws;
        next.active_idx = nx->active_idx;
        next.n_active = nx->n_active;
        next.n_found = nx->n_found;
        next.target_pos = nx->target_pos;
        next.dev_status = dev_status;
    }
    rc = sm_run(W_bf16, X_bf16, D, B, M, scale, grad_scale, active_idx, n_active, target_pos, loss_per_sample, loss_mean, dX,
                dW_active, s.w, flags, dev_status, st, nullptr, SM_IMPORT, io, DwUpdate(), ride ? &next : nullptr);
    if (rc == KS_OK && nx && !ride)
        rc = knn_select_active_csr(nx->labels, nx->counts, nx->offsets, nx->flat, nx->flat_len, nx->Cg, nx->c0, C, B, nx->K_max, M,
                                   nx->sel_flags, nx->pad_seed, nx->active_idx, nx->n_active, nx->n_found, nx->target_pos, sel_ws,
                                   ks_select_ws_bytes(C, B, nx->K_max), dev_status, stream);
    return rc;
}
extern "C" int knn_softmax_bwd_from_stats(const uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *active_idx,
                                          const int32_t *n_active, const int32_t *target_pos, const float *global_max,
                                          const float *global_sumexp, const float *global_target_logit, int64_t C, int D,
                                          int B, int M, float scale, float grad_scale, uint32_t flags,
                                          float *loss_per_sample, float *loss_mean, float *dX, float *dW_active, void *ws,
                                          size_t ws_bytes, int32_t *dev_status, void *stream) {
    return sm_bwd_from_stats(W_bf16, X_bf16, active_idx, n_active, target_pos, global_max, global_sumexp, global_target_logit,
                             C, D, B, M, scale, grad_scale, flags, loss_per_sample, loss_mean, dX, dW_active, nullptr, ws,
                             ws_bytes, dev_status, stream);
}
extern "C" size_t knn_softmax_split_next_workspace(int64_t C, int D, int B, int K_max, int M) {
    if (sm_split_check(C, D, B, M, 1.f, 0) != KS_OK || K_max < 0) return 0;
    size_t total = 0;
    sm_split_carve(nullptr, C, D, B, M, true, &total);
    return ks_align_up(total, 256) + ks_select_ws_bytes(C, B, K_max);
}
extern "C" int knn_softmax_bwd_from_stats_next(const uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *active_idx,
                                               const int32_t *n_active, const int32_t *target_pos, const float *global_max,
                                               const float *global_sumexp, const float *global_target_logit, int64_t C, int D,
                                               int B, int M, float scale, float grad_scale, uint32_t flags,
                                               float *loss_per_sample, float *loss_mean, float *dX, float *dW_active,
                                               const int32_t *labels_next, const int32_t *counts, const int64_t *offsets,
                                               const int32_t *flat, int64_t flat_len, int64_t Cg, int64_t c0, int K_max,
                                               uint32_t select_flags, uint64_t pad_seed, int32_t *active_idx_next,
                                               int32_t *n_active_next, int32_t *n_found_next, int32_t *target_pos_next,
                                               void *ws, size_t ws_bytes, int32_t *dev_status, void *stream) {
    SmNextCsr nx{labels_next, counts, offsets, flat, flat_len, Cg, c0, K_max, select_flags, pad_seed, active_idx_next,
                 n_active_next, n_found_next, target_pos_next};
    return sm_bwd_from_stats(W_bf16, X_bf16, active_idx, n_active, target_pos, global_max, global_sumexp, global_target_logit,
                             C, D, B, M, scale, grad_scale, flags, loss_per_sample, loss_mean, dX, dW_active, &nx, ws, ws_bytes,
                             dev_status, stream);
}

// The step on a selection computed earlier (possibly on another stream): sanitised copy of the list, then everything
// after the selection.  The softmax buffers come first in the workspace, the copy of the list after them.
static int sm_selected_check(int64_t C, int D, int B, int M) {
    if (sm_check_dims(C, D, B) != KS_OK || M < 1 || B > M) return KS_INVALID_ARG;
    return KS_OK;
}
extern "C" size_t knn_softmax_selected_workspace(int64_t C, int D, int B, int M) {
    if (sm_selected_check(C, D, B, M) != KS_OK) return 0;
    size_t total = 0;
    sm_split_carve(nullptr, C, D, B, M, true, &total);
    return sm_with_kept(total, B, D, M);
}
// the next batch's selection that rides along with a step on a given selection (nullptr: none)
struct SmNextArgs {
    const int32_t *labels, *graph;
    int K;
    int32_t *active_idx, *n_active, *target_pos;
};
static int sm_selected(float *W_master, uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *active_idx,
                       const int32_t *n_active, const int32_t *target_pos, int64_t C, int D, int B, int M, float scale,
                       float grad_scale, float alpha, uint32_t flags, float *loss_per_sample, float *loss_mean, float *dX,
                       float *dW_active, const SmNextArgs *nx, void *ws, size_t ws_bytes, int32_t *dev_status, void *stream) {
    if (!W_bf16 || !X_bf16 || !active_idx || !n_active || !target_pos || !loss_per_sample || !loss_mean || !dX || !ws)
        return KS_INVALID_ARG;
    if (sm_selected_check(C, D, B, M) != KS_OK) return KS_INVALID_ARG;
    if (flags & ~(uint32_t)(KS_FLAG_UNIT_ROWS | KS_FLAG_TRUSTED_LIST)) return KS_INVALID_ARG;
    const bool fast = sm_fast(D, B, scale, grad_scale);
    const bool trusted = (flags & KS_FLAG_TRUSTED_LIST) != 0;
    if (!dW_active && !(W_master && D % 64 == 0)) return KS_INVALID_ARG;
    // a trusted list is read where it lies, until the end of the call: the next batch's list needs buffers of its own
    if (nx && trusted && (nx->active_idx == active_idx || nx->n_active == n_active || nx->target_pos == target_pos))
        return KS_INVALID_ARG;
    if (nx) {
        if (!nx->labels || !nx->active_idx || !nx->n_active || !nx->target_pos || nx->K < 0 || (nx->K > 0 && !nx->graph))
            return KS_INVALID_ARG;
        if ((int64_t)nx->K + 1 > M) return KS_INVALID_ARG;
    }
    size_t need = 0;
    SmSplitWs s = sm_split_carve(ws, C, D, B, M, fast, &need);
    if (nx) need = ks_align_up(need, 256);
    void *sel_ws = (char *)ws + need; // the selection's staging area follows the step's buffers
    if (nx) need += ks_select_ws_bytes(C, B, nx->K);
    if (ws_bytes < need) return KS_WORKSPACE_TOO_SMALL;
    sm_take_kept(s.w, ws, need, ws_bytes, B, D, M);
    hipStream_t st = (hipStream_t)stream;
    const int nmax = M > B ? M : B;
    const int32_t *act = active_idx, *n_act = n_active, *tp = target_pos;
    if (!trusted) { // the validated copy (which also lets the next batch's list be written where this one came in)
        hipLaunchKernelGGL(sm_sanitize_kernel, dim3((unsigned)ks_ceil_div(nmax, SM_NT)), dim3(SM_NT), 0, st, active_idx,
                           n_active, target_pos, C, M, B, s.act, s.n, s.tp, dev_status);
        act = s.act;
        n_act = s.n;
        tp = s.tp;
    }
    DwUpdate up = DwUpdate();
    if (W_master && fast) {
        up.Wm = W_master;
        up.Wb = W_bf16;
        up.idx = act;
        up.alpha = alpha;
    }
    // The selection rides along with the dX and dW launches of the fast path where the class bitmap fits in LDS; otherwise it
    // follows the step as launches of its own.  Either way it starts after the sanitised copy
    // of this step's list has been made, so its outputs may be the buffers this step's list came in.
    KsSelNext next = KsSelNext();
    const bool ride = nx && fast && sm_next_rides(C, B, nx->K);
    if (ride) {
        next.nsel = SEL1_GRID;
        next.dense = SelDense{nx->labels, nx->graph, C, nx->K};
        next.pad = sel_pad_make(0, C, 0);
        next.C = C;
        next.B = B;
        next.K = nx->K;
        next.M = M;
        next.cand = (int32_t *)sel_ws;
        next.active_idx = nx->active_idx;
        next.n_active = nx->n_active;
        next.target_pos = nx->target_pos;
        next.dev_status = dev_status;
    }
    int rc = sm_run(W_bf16, X_bf16, D, B, M, scale, grad_scale, act, n_act, tp, loss_per_sample, loss_mean, dX, dW_active,
                    s.w, flags & KS_FLAG_UNIT_ROWS, dev_status, st, nullptr, SM_WHOLE, SmSplitIO(), up, ride ? &next : nullptr);
    if (rc == KS_OK && W_master && !fast)
        rc = apply_weight_grad(W_master, W_bf16, act, n_act, M, dW_active, alpha, C, D, 1, ws, ws_bytes, dev_status, stream);
    if (rc == KS_OK && nx && !ride)
        rc = ks_select_launch(nx->labels, nx->graph, C, B, nx->K, M, nx->active_idx, nx->n_active, nx->target_pos, sel_ws,
                              dev_status, st);
    return rc;
}
extern "C" int knn_softmax_fwd_bwd_update_selected(float *W_master, uint16_t *W_bf16, const uint16_t *X_bf16,
                                                   const int32_t *active_idx, const int32_t *n_active,
                                                   const int32_t *target_pos, int64_t C, int D, int B, int M, float scale,
                                                   float grad_scale, float alpha, uint32_t flags, float *loss_per_sample,
                                                   float *loss_mean, float *dX, float *dW_active, void *ws, size_t ws_bytes,
                                                   int32_t *dev_status, void *stream) {
    return sm_selected(W_master, W_bf16, X_bf16, active_idx, n_active, target_pos, C, D, B, M, scale, grad_scale, alpha, flags,
                       loss_per_sample, loss_mean, dX, dW_active, nullptr, ws, ws_bytes, dev_status, stream);
}
extern "C" size_t knn_softmax_selected_next_workspace(int64_t C, int D, int B, int K, int M) {
    if (sm_selected_check(C, D, B, M) != KS_OK || K < 0) return 0;
    size_t total = 0;
    sm_split_carve(nullptr, C, D, B, M, true, &total);
    return sm_with_kept(ks_align_up(total, 256) + ks_select_ws_bytes(C, B, K), B, D, M);
}
extern "C" int knn_softmax_fwd_bwd_update_selected_next(float *W_master, uint16_t *W_bf16, const uint16_t *X_bf16,
                                                        const int32_t *active_idx, const int32_t *n_active,
                                                        const int32_t *target_pos, int64_t C, int D, int B, int M,
                                                        float scale, float grad_scale, float alpha, uint32_t flags,
                                                        float *loss_per_sample, float *loss_mean, float *dX,
                                                        float *dW_active, const int32_t *labels_next, const int32_t *graph,
                                                        int K, int32_t *active_idx_next, int32_t *n_active_next,
                                                        int32_t *target_pos_next, void *ws, size_t ws_bytes,
                                                        int32_t *dev_status, void *stream) {
    SmNextArgs nx{labels_next, graph, K, active_idx_next, n_active_next, target_pos_next};
    return sm_selected(W_master, W_bf16, X_bf16, active_idx, n_active, target_pos, C, D, B, M, scale, grad_scale, alpha, flags,
                       loss_per_sample, loss_mean, dX, dW_active, &nx, ws, ws_bytes, dev_status, stream);
}

static size_t full_bytes(int64_t C, int D, int B) {
    return sm_bytes(C, D, B, 0, C, false) + ks_align_up((size_t)C * 4, 256) + ks_align_up((size_t)B * 4, 256) + 256;
}
extern "C" size_t full_softmax_workspace(int64_t C, int D, int B) {
    if (sm_check_dims(C, D, B) != KS_OK) return 0;
    return sm_with_kept(full_bytes(C, D, B), B, D, C);
}

extern "C" int full_softmax_fwd_bwd(const uint16_t *W_bf16, const uint16_t *X_bf16, const int32_t *labels, int64_t C,
                                    int D, int B, float scale, float grad_scale, uint32_t flags, float *loss_per_sample,
                                    float *loss_mean, float *dX, float *dW, void *ws, size_t ws_bytes,
                                    int32_t *dev_status, void *stream) {
    if (!W_bf16 || !X_bf16 || !labels || !loss_per_sample || !loss_mean || !dX || !dW || !ws) return KS_INVALID_ARG;
    if (sm_check_dims(C, D, B) != KS_OK) return KS_INVALID_ARG;
    const size_t need = full_bytes(C, D, B);
    if (ws_bytes < need) return KS_WORKSPACE_TOO_SMALL;
    SmWs w = sm_carve(ws, C, D, B, 0, C, false, sm_fast(D, B, scale, grad_scale));
    sm_take_kept(w, ws, need, ws_bytes, B, D, C);
    KsArena ar((char *)ws + sm_bytes(C, D, B, 0, C, false));
    int32_t *active_idx = ar.take<int32_t>((size_t)C);
    int32_t *target_pos = ar.take<int32_t>((size_t)B);
    int32_t *n_active = ar.take<int32_t>(1);
    hipStream_t st = (hipStream_t)stream;
    int64_t n = C > B ? C : B;
    hipLaunchKernelGGL(full_prepare_kernel, dim3((unsigned)ks_ceil_div(n, SM_NT)), dim3(SM_NT), 0, st, labels, C, B,
                       active_idx, n_active, target_pos, dev_status);
    return sm_run(W_bf16, X_bf16, D, B, C, scale, grad_scale, active_idx, n_active, target_pos, loss_per_sample,
                  loss_mean, dX, dW, w, flags, dev_status, st);
}

extern "C" int knn_gather_rows(const uint16_t *W_bf16, const int32_t *active_idx, const int32_t *n_active, int M,
                               int64_t C, int D, uint16_t *out, int32_t *dev_status, void *stream) {
    if (!W_bf16 || !active_idx || !n_active || !out) return KS_INVALID_ARG;
    if (M < 1 || C < 1 || D < 8 || D % 8 != 0) return KS_INVALID_ARG;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)ks_ceil_div(M, SM_NT / 64)), dim3(SM_NT), 0, (hipStream_t)stream,
                       W_bf16, active_idx, n_active, M, C, D, out, dev_status);
    KS_LAUNCH_CHECK();
    return KS_OK;
}

extern "C" const char *ks_version(void) { return "knnsoftmax 0.1 (gfx950)"; }
