// Learning-to-hash trainer: one SGD step on the hash weights of one attention head (Sec. 3.1 of
// the paper, the final multi-query hashing model; App. B.2 for the optimiser).
//
//   L = c_sim sum_n s_n ||h(q_n) - h(k_n)||^2 + c_bal sum_j ||sum_{n in query j} h(k_n)||^2
//       + lam ||W^T W - I||_F,      h(x) = 2 Sigmoid(sigma x W) - 1 = tanh(sigma x W / 2)
// (the balance term per query j, as the final hashing model prints it: the triplets of a query fill
// whole blocks of TR_ROWS rows and every block names its query; without names the batch is one query)
//
// The two projections X W ([n,128] x [128,r]) and the weight-gradient contraction X^T dZ
// ([128,n] x [n,r]) are dense contractions and run on MFMA (v_mfma_f32_32x32x16_bf16).  q and k are
// bf16 already; fp32 operands (W, dZ) are split exactly into three bf16 planes, so every product is
// exact and only the fp32 accumulation rounds.
//
// Launches of a step (three, four for batches of more than TR_FEW_WGS blocks):
//   1. train_colsum_kernel   h(k) of every key -> per-workgroup column sums (the balance term couples
//                            every row to the sum of h(k) over its query, so those sums come first);
//                            extra workgroups: P = W^T W - I and its squared Frobenius norm, and the
//                            three bf16 planes of W in operand order for the next launch
//      (train_colreduce_kernel adds the column sums up per query when there are too many workgroups
//      for every workgroup of the next launch to do so for its own query)
//   2. train_grad_kernel     forward of q and k again, dL/dz elementwise in the MFMA result
//                            registers, then X^T dZ with those registers as the B operand (the
//                            contraction index -- the row -- may be enumerated in any order, so the
//                            32x32 result layout is used as it stands; only X is read transposed,
//                            from the LDS tile it was staged in) -> per-workgroup partial dW;
//                            extra workgroups: W P
//   3. train_update_kernel   dL/dW = sigma sum partials + 2 lam W P / ||P||_F, the loss terms, weight
//                            decay, momentum, step
// What does not depend on a launch's main work rides along in extra workgroups of it, so that the chain is
// as short as the data flow allows: at r = 128 and 32768 triplets six launches took 63 us of kernel time a step, the
// three take 37 us.
#include <new>

#include "hata_device.h"
#include "../../include/hata_train.h"

struct LabelCand { unsigned long long key; uint32_t row, pad; };

struct hata_train_ctx {
    hata_train_config cfg;
    int n_wgs_max;
    float* colsum_part;  // [n_wgs_max, r]
    float* colsum;       // [queries (<= n_wgs_max), r]  sum of h(k_n) over the triplets of a query
    float* bal_part;     // [column groups (<= 2), n_wgs_max]  squared norms of those sums, a query's at its first workgroup
    float* dw_part;      // [n_wgs_max, d, r]
    float* loss_part;    // [column groups (<= 2), n_wgs_max]
    float* P;            // [r, r]
    float* fro_part;     // [r]
    float* WP;           // [d, r]  W (W^T W - I)
    uint4* planes;       // [r / 32, 3, 8, 64]  bf16 planes of W as operand fragments, 16 bytes a lane
    // label builder
    double* scores;      // [n_max] qk scores
    uint32_t* bins;      // [LB_COPIES, LB_BINS] how many scores fall into each bin, zero between calls
    int bins_clear;      // a label call has left them so (the first one clears them on its own stream)
    uint32_t* n_cand;    // [1] entries of the candidate list
    LabelCand* cand;     // [n_max]
};

namespace hata {

typedef __attribute__((ext_vector_type(8))) __bf16 tr_bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float tr_f32x16_t;
#define TR_ROWS 128   // triplets per workgroup (one LDS stage)
#define TR_FEW_WGS 512  // up to here every workgroup of the gradient launch sums its query's column sums itself
#define TR_PITCH 136  // LDS row pitch in bf16 elements (272 B: conflict-free 16-B and transposed reads)

// Two fp32 values -> three bf16 terms each, whose sum carries all 24 mantissa bits (each term is the
// remainder truncated to its upper 8 significant bits, so both subtractions are exact); the pair's terms are packed
// into a dword each
__device__ __forceinline__ uint32_t pack_hi16(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
__device__ __forceinline__ void split3_pair(float x0, float x1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    const uint32_t h0 = __float_as_uint(x0) & 0xffff0000u, h1 = __float_as_uint(x1) & 0xffff0000u;
    const float r0 = x0 - __uint_as_float(h0), r1 = x1 - __uint_as_float(h1);
    const uint32_t m0 = __float_as_uint(r0) & 0xffff0000u, m1 = __float_as_uint(r1) & 0xffff0000u;
    hi = pack_hi16(h0, h1);
    mid = pack_hi16(m0, m1);
    lo = pack_hi16(__float_as_uint(r0 - __uint_as_float(m0)), __float_as_uint(r1 - __uint_as_float(m1)));
}

// h = 2 Sigmoid(sigma z) - 1, with nsl = -sigma log2(e)
__device__ __forceinline__ float relaxed_sign(float z, float nsl) {
    return fmaf(2.f, __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(nsl * z)), -1.f);
}
#define TR_LOG2E 1.4426950408889634f

// Weight fragments of hash column `col` as the B operand:
// frag[plane][kk] holds W[16 kk + 8 half + e][col], e = 0..7
template <int R>
__device__ __forceinline__ void load_weight_planes(const float* __restrict__ W, int col, int half,
                                                   tr_bf16x8_t (&frag)[3][8]) {
    const float* wp = W + col;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        uint32_t hi[4], mid[4], lo[4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            const float* w2 = wp + (int64_t)(kk * 16 + 8 * half + 2 * e2) * R;
            split3_pair(w2[0], w2[R], hi[e2], mid[e2], lo[e2]);
        }
        frag[0][kk] = __builtin_bit_cast(tr_bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
        frag[1][kk] = __builtin_bit_cast(tr_bf16x8_t, make_uint4(mid[0], mid[1], mid[2], mid[3]));
        frag[2][kk] = __builtin_bit_cast(tr_bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
    }
}

// How a workgroup's waves share its TR_ROWS rows and up to 128 hash columns: a wave owns 32 columns and
// 1 / RS of the rows (RS = row split).  At least two waves per SIMD where the columns allow it: with one,
// nothing covers the exponentials and LDS reads between its matrix instructions.
template <int R>
struct TrainShape {
    static constexpr int COLS = R < 128 ? R : 128;  // columns of a workgroup
    static constexpr int CG = COLS / 32;
    static constexpr int RS = CG == 4 ? 2 : 4;
    static constexpr int THREADS = CG * RS * 64;
    static constexpr int TILES = TR_ROWS / 32 / RS;  // 32-row tiles of a wave
    static constexpr int WAVES = THREADS / 64;
    static constexpr int SLICES = THREADS / COLS;  // threads per column (below 64 columns more than the waves)
    static constexpr int COL_ROWS = WAVES > SLICES ? WAVES : SLICES;  // rows of LDS that per-column sums of either kind need
};

// rows [row0, row0 + TR_ROWS) of X [n, 128] (zeros past n): fetched into registers, later put into an LDS tile
template <int THREADS>
struct StagedRows {
    static constexpr int NV = TR_ROWS * 16 / THREADS;
    uint4 v[NV];
    __device__ __forceinline__ void fetch(const uint16_t* __restrict__ X, int row0, int n) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = threadIdx.x + j * THREADS, row = i >> 4, sub = i & 15;
            v[j] = make_uint4(0, 0, 0, 0);
            if (row0 + row < n) v[j] = *reinterpret_cast<const uint4*>(X + (int64_t)(row0 + row) * HATA_D + sub * 8);
        }
    }
    __device__ __forceinline__ void put(uint16_t* tile) const {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = threadIdx.x + j * THREADS, row = i >> 4, sub = i & 15;
            *reinterpret_cast<uint4*>(&tile[row * TR_PITCH + sub * 8]) = v[j];
        }
    }
};

// Z tile t (32 rows x the wave's 32 columns) = X_tile . W: result register ri of lane (m, half)
// holds row 8 (ri / 4) + 4 half + ri % 4 of the tile, column 32 w + m
__device__ __forceinline__ tr_f32x16_t project_tile(const uint16_t* tile, int t, int m, int half,
                                                    const tr_bf16x8_t (&wfrag)[3][8]) {
    tr_f32x16_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        const tr_bf16x8_t x = *reinterpret_cast<const tr_bf16x8_t*>(&tile[(t * 32 + m) * TR_PITCH + kk * 16 + 8 * half]);
#pragma unroll
        for (int p = 0; p < 3; ++p) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, wfrag[p][kk], acc, 0, 0, 0);
    }
    return acc;
}

// Channel step kk of the fragments of 32 hash columns into the workspace (one wave), and all of them back
template <int R>
__device__ __forceinline__ void store_weight_planes(const float* __restrict__ W, int cgroup, int kk, uint4* __restrict__ planes) {
    const int lane = threadIdx.x & 63;
    const float* wp = W + (int64_t)(kk * 16 + 8 * (lane >> 5)) * R + cgroup * 32 + (lane & 31);
    uint32_t f[3][4];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2)
        split3_pair(wp[(int64_t)(2 * e2) * R], wp[(int64_t)(2 * e2 + 1) * R], f[0][e2], f[1][e2], f[2][e2]);
#pragma unroll
    for (int p = 0; p < 3; ++p)
        planes[((cgroup * 3 + p) * 8 + kk) * 64 + lane] = make_uint4(f[p][0], f[p][1], f[p][2], f[p][3]);
}
__device__ __forceinline__ void fetch_weight_planes(const uint4* __restrict__ planes, int cgroup, tr_bf16x8_t (&frag)[3][8]) {
    const uint4* src = planes + cgroup * 3 * 8 * 64 + (threadIdx.x & 63);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
#pragma unroll
        for (int p = 0; p < 3; ++p) frag[p][kk] = __builtin_bit_cast(tr_bf16x8_t, src[(p * 8 + kk) * 64]);
}

// P = W^T W - I (column j by one workgroup) and the squared Frobenius norm of that column; THREADS threads,
// red: THREADS / 64 floats of LDS
template <int THREADS>
__device__ __forceinline__ void gram_column(const float* __restrict__ W, int r, int j, float* __restrict__ P,
                                            float* __restrict__ fro_part, float* red) {
    const int tid = threadIdx.x;
    float sq = 0.f;
    for (int i = tid; i < r; i += THREADS) {
        float acc = 0.f;
#pragma unroll 16
        for (int c = 0; c < HATA_D; ++c) acc = fmaf(W[(int64_t)c * r + i], W[(int64_t)c * r + j], acc);
        acc -= (i == j) ? 1.f : 0.f;
        P[(int64_t)i * r + j] = acc;
        sq = fmaf(acc, acc, sq);
    }
    sq = wave_sum64(sq);
    if ((tid & 63) == 0) red[tid >> 6] = sq;
    __syncthreads();
    if (tid == 0) {
        float t = 0.f;
        for (int i = 0; i < THREADS / 64; ++i) t += red[i];
        fro_part[j] = t;
    }
}

// grid = (n_wgs workgroups of TR_ROWS triplets, then eight for the group's weight planes, then one for each of
// its columns of the Gram matrix; groups of up to 128 hash columns)
template <int R>
__global__ __launch_bounds__(TrainShape<R>::THREADS) void train_colsum_kernel(
    const uint16_t* __restrict__ K, const float* __restrict__ W, int n, int n_wgs, float sigma,
    float* __restrict__ colsum_part, float* __restrict__ P, float* __restrict__ fro_part, uint4* __restrict__ planes) {
    using S = TrainShape<R>;
    __shared__ __attribute__((aligned(16))) uint16_t tile[TR_ROWS * TR_PITCH];
    __shared__ float s_part[S::RS][S::COLS];
    if ((int)blockIdx.x >= n_wgs) {
        const int j = (int)blockIdx.x - n_wgs - 8;
        if (j >= 0) gram_column<S::THREADS>(W, R, blockIdx.y * S::COLS + j, P, fro_part, &s_part[0][0]);
        else if (threadIdx.x < S::CG * 64) store_weight_planes<R>(W, blockIdx.y * 4 + threadIdx.x / 64, j + 8, planes);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, w = (tid >> 6) % S::CG, rs = (tid >> 6) / S::CG;
    const int m = lane & 31, half = lane >> 5;
    const int col = blockIdx.y * 128 + w * 32 + m;
    StagedRows<S::THREADS> xk;
    xk.fetch(K, blockIdx.x * TR_ROWS, n);
    tr_bf16x8_t wfrag[3][8];
    load_weight_planes<R>(W, col, half, wfrag);
    xk.put(tile);
    __syncthreads();
    const float nsl = -sigma * TR_LOG2E;
    float cs = 0.f;
#pragma unroll
    for (int t = 0; t < S::TILES; ++t) {
        const tr_f32x16_t z = project_tile(tile, rs * S::TILES + t, m, half, wfrag);
#pragma unroll
        for (int i = 0; i < 16; ++i) cs += relaxed_sign(z[i], nsl);  // (rows past n are zero: h = 0)
    }
    cs += __shfl_xor(cs, 32, 64);
    if (half == 0) s_part[rs][w * 32 + m] = cs;
    __syncthreads();
    if (tid < S::COLS) {
        float t = s_part[0][tid];
#pragma unroll
        for (int i = 1; i < S::RS; ++i) t += s_part[i][tid];
        colsum_part[(int64_t)blockIdx.x * R + blockIdx.y * 128 + tid] = t;
    }
}

// the query a block of TR_ROWS triplets belongs to (no names: everything is query 0; a name outside
// [0, n_groups) counts as the nearest valid one, so no access leaves the arrays)
__device__ __forceinline__ int block_query(const int32_t* __restrict__ block_group, int wg, int n_groups) {
    return block_group ? clampi(block_group[wg], 0, n_groups - 1) : 0;
}

// sum of the per-workgroup column sums of one query: one workgroup per (hash column, query)
__global__ __launch_bounds__(256) void train_colreduce_kernel(const float* __restrict__ colsum_part, int r,
                                                              int n_wgs, const int32_t* __restrict__ block_group,
                                                              int n_groups, float* __restrict__ colsum) {
    __shared__ float red[4];
    const int j = blockIdx.x, q = blockIdx.y, tid = threadIdx.x;
    float acc = 0.f;
    for (int g = tid; g < n_wgs; g += 256)
        if (block_query(block_group, g, n_groups) == q) acc += colsum_part[(int64_t)g * r + j];
    acc = wave_sum64(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) colsum[(int64_t)q * r + j] = red[0] + red[1] + red[2] + red[3];
}

// Four rows of one channel per lane, from an LDS tile of rows: every group of 16 lanes reads 4 rows x 16
// channels (lane: 8 bytes of row lane % 16 / 4) and gets them transposed (lane: channel lane % 16, the four
// rows).  p: where this lane reads.
typedef __attribute__((ext_vector_type(4))) short tr_s16x4_t;
__device__ __forceinline__ uint2 lds_read_transposed(const uint16_t* p) {
    const tr_s16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) tr_s16x4_t*)(uint16_t*)p);
    return __builtin_bit_cast(uint2, v);
}

// grid = (n_wgs blocks of TR_ROWS triplets and then 128 workgroups for the rows of W P, column groups).
// colsum: per-query sums (train_colreduce_kernel), or nullptr: this workgroup adds its query's up itself
// from colsum_part and leaves their squared norm in bal_part if it is the query's first.
//
// What bounds it: one round of workgroups, so the latency of what a workgroup reads (rows, weight planes,
// column sums: 8 us until the first matrix instruction, 4 of them the column sums) and then, added up, the
// matrix instructions (96 per 32-row tile and wave: two projections of three planes, two contractions of
// three) and the exponentials (11 us).  Hence eight waves per workgroup, two per SIMD; the planes made once,
// by the launch before, instead of split from W in every workgroup; transposing LDS reads instead of 2-byte
// ones: 31 -> 25 us at r = 128 and 32768 triplets, the sums of the old reduction launch (4.4 us) included.
template <int R>
__global__ __launch_bounds__(TrainShape<R>::THREADS) void train_grad_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const float* __restrict__ s,
    const float* __restrict__ W, const uint4* __restrict__ planes, int n, int n_wgs, float sigma, float c_sim,
    float c_bal, const float* __restrict__ colsum, const float* __restrict__ colsum_part, const int32_t* __restrict__ block_group,
    int n_groups, const float* __restrict__ P, float* __restrict__ dw_part, float* __restrict__ loss_part,
    float* __restrict__ bal_part, float* __restrict__ WP) {
    using S = TrainShape<R>;
    constexpr int THREADS = S::THREADS, WAVES = S::WAVES, SLICES = S::SLICES;
    __shared__ __attribute__((aligned(16))) uint16_t tile[2 * TR_ROWS * TR_PITCH];
    __shared__ float s_lab[TR_ROWS];
    __shared__ __attribute__((aligned(16))) float s_col[S::COL_ROWS][S::COLS];  // per hash column: sums of h(k_n) over this block's query, a wave's each; or of a row of W P, a slice's each
    static_assert(sizeof(s_col) >= sizeof(float) * S::COLS * (WAVES > SLICES ? WAVES : SLICES), "a row per wave, and per slice");
    __shared__ float s_bal[WAVES], s_loss[WAVES];
    __shared__ int s_first;
    const int tid = threadIdx.x, lane = tid & 63;
    const int jc = tid % S::COLS, sl = tid / S::COLS;
    if ((int)blockIdx.x >= n_wgs) {  // row c of W P
        const int c = blockIdx.x - n_wgs, j = blockIdx.y * 128 + jc;
        const int i0 = sl * (R / SLICES);
        float wp = 0.f;
#pragma unroll 16
        for (int i = i0; i < i0 + R / SLICES; ++i) wp = fmaf(W[(int64_t)c * R + i], P[(int64_t)i * R + j], wp);
        s_col[sl][jc] = wp;
        __syncthreads();
        if (sl == 0) {
#pragma unroll
            for (int i = 1; i < SLICES; ++i) wp += s_col[i][jc];
            WP[(int64_t)c * R + j] = wp;
        }
        return;
    }
    uint16_t* const tile_q = tile;
    uint16_t* const tile_k = tile + TR_ROWS * TR_PITCH;
    const int w = (tid >> 6) % S::CG, rs = (tid >> 6) / S::CG;
    const int m = lane & 31, half = lane >> 5;
    const int row0 = blockIdx.x * TR_ROWS;
    const int col = blockIdx.y * 128 + w * 32 + m;
    // everything the workgroup reads is requested before anything is waited for
    StagedRows<THREADS> xq, xk;
    xq.fetch(Q, row0, n);
    xk.fetch(K, row0, n);
    tr_bf16x8_t wfrag[3][8];
    fetch_weight_planes(planes, blockIdx.y * 4 + w, wfrag);
    if (tid == 0) s_first = 1;
    for (int i = tid; i < TR_ROWS; i += THREADS) s_lab[i] = (row0 + i < n) ? s[row0 + i] : 0.f;
    // the column sums of this block's query
    const int query = block_query(block_group, blockIdx.x, n_groups);
    if (colsum) {
        if (sl == 0) s_col[0][jc] = colsum[(int64_t)query * R + blockIdx.y * 128 + jc];
        xq.put(tile_q);
        xk.put(tile_k);
    } else {
        // a wave takes a run of blocks, whole rows of column sums at a time: which of them are this
        // query's is the same for all its lanes (scalar loads and branches)
        constexpr int NV = S::COLS > 64 ? 2 : 1;
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), per = (n_wgs + WAVES - 1) / WAVES;
        const int g0 = wv * per, g1 = min(n_wgs, g0 + per), j0 = lane * NV;
        const float* cp = colsum_part + blockIdx.y * 128 + min(j0, S::COLS - NV);
        float sum[NV] = {};
        bool earlier = false;
        for (int g = g0; g < g1; g += 32) {
            float x[32][NV];
#pragma unroll
            for (int u = 0; u < 32; ++u)
#pragma unroll
                for (int e = 0; e < NV; ++e) x[u][e] = cp[(int64_t)min(g + u, g1 - 1) * R + e];
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                const bool own = g + u < g1 && block_query(block_group, min(g + u, g1 - 1), n_groups) == query;
                earlier |= own && g + u < (int)blockIdx.x;
#pragma unroll
                for (int e = 0; e < NV; ++e) sum[e] += own ? x[u][e] : 0.f;
            }
        }
        xq.put(tile_q);
        xk.put(tile_k);
        if (j0 < S::COLS) {
#pragma unroll
            for (int e = 0; e < NV; ++e) s_col[wv][j0 + e] = sum[e];
        }
        __syncthreads();
        if (lane == 0 && earlier) s_first = 0;
        float t = 0.f;
        if (tid < S::COLS) {
#pragma unroll
            for (int i = 0; i < WAVES; ++i) t += s_col[i][tid];
            s_col[0][tid] = t;  // (read by this thread alone before)
        }
        __syncthreads();
        t = wave_sum64(s_first ? t * t : 0.f);
        if (lane == 0) s_bal[tid >> 6] = t;
    }
    __syncthreads();
    if (tid == 0 && !colsum) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) t += s_bal[i];
        bal_part[blockIdx.y * n_wgs + blockIdx.x] = t;
    }
    const float nsl = -sigma * TR_LOG2E, colk = c_bal * s_col[0][w * 32 + m];
    tr_f32x16_t dw[4];  // dw[ct][ri]: channel 32 ct + 8 (ri / 4) + 4 half + ri % 4, this lane's column
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) dw[ct][i] = 0.f;
    float lsim = 0.f;
    // where this lane reads of a 4-row x 16-channel piece of a tile (lds_read_transposed), for row group
    // 4 half and channel group 16 (m / 16)
    const int tr_off = (4 * half + (lane & 15) / 4) * TR_PITCH + 16 * (m >> 4) + 4 * (lane & 3);
#pragma unroll 1
    for (int tt = 0; tt < S::TILES; ++tt) {
        const int t = rs * S::TILES + tt;
        tr_f32x16_t zq = project_tile(tile_q, t, m, half, wfrag);  // then dL/dz of q
        tr_f32x16_t zk = project_tile(tile_k, t, m, half, wfrag);  // then dL/dz of k
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = t * 32 + 8 * (i / 4) + 4 * half + (i % 4);
            const float hq = relaxed_sign(zq[i], nsl), hk = relaxed_sign(zk[i], nsl);
            const float diff = hq - hk, sd = s_lab[row] * diff;
            const float dhq = c_sim * sd, dhk = colk - dhq;  // (half of dL/dh: h' = (1 - h^2) / 2)
            zq[i] = dhq * fmaf(-hq, hq, 1.f);
            zk[i] = dhk * fmaf(-hk, hk, 1.f);
            lsim = fmaf(sd, diff, lsim);
        }
        // X^T dZ over the tile's 32 rows, 16 per MFMA: the B operand is dZ as it sits in the
        // registers (slot (half, j) of step ks <-> row 16 ks + 8 (j / 4) + 4 half + j % 4), the A
        // operand X read from the LDS tile in that same row order
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int qk = 0; qk < 2; ++qk) {
                const uint16_t* tl = (qk ? tile_k : tile_q) + (t * 32 + 16 * ks) * TR_PITCH + tr_off;
                tr_bf16x8_t bz[3];
                {
                    uint32_t pz[3][4];
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2) {
                        const int i = 8 * ks + 2 * e2;
                        split3_pair(qk ? zk[i] : zq[i], qk ? zk[i + 1] : zq[i + 1], pz[0][e2], pz[1][e2], pz[2][e2]);
                    }
#pragma unroll
                    for (int p = 0; p < 3; ++p)
                        bz[p] = __builtin_bit_cast(tr_bf16x8_t, make_uint4(pz[p][0], pz[p][1], pz[p][2], pz[p][3]));
                }
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) {
                    const uint2 lo = lds_read_transposed(tl + 32 * ct), hi = lds_read_transposed(tl + 32 * ct + 8 * TR_PITCH);
                    const tr_bf16x8_t x = __builtin_bit_cast(tr_bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
                    for (int p = 0; p < 3; ++p) dw[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, bz[p], dw[ct], 0, 0, 0);
                }
            }
        }
    }
    lsim = wave_sum64(lsim);
    if (lane == 0) s_loss[tid >> 6] = lsim;
    // the row groups' partial sums of a column group meet in the tiles' LDS, halving each time
    float* const meet = reinterpret_cast<float*>(tile);
#pragma unroll
    for (int rows = S::RS / 2; rows >= 1; rows >>= 1) {
        static_assert(S::RS / 2 * S::CG * 64 * 64 * 4 <= (int)sizeof(tile), "the sums of half the row groups fit");
        __syncthreads();
        float* mp = meet + (int64_t)((rs % rows) * S::CG + w) * 64 * 64 + lane;
        if (rs >= rows && rs < 2 * rows) {
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int i = 0; i < 16; ++i) mp[(ct * 16 + i) * 64] = dw[ct][i];
        }
        __syncthreads();
        if (rs < rows) {
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int i = 0; i < 16; ++i) dw[ct][i] += mp[(ct * 16 + i) * 64];
        }
    }
    if (rs == 0) {
        float* out = dw_part + (int64_t)blockIdx.x * HATA_D * R;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int ch = 32 * ct + 8 * (i / 4) + 4 * half + (i % 4);
                out[(int64_t)ch * R + col] = dw[ct][i];
            }
    }
    if (tid == 0) {  // (the similarity partial of column group y; the groups are summed later)
        float t = 0.f;
        for (int i = 0; i < WAVES; ++i) t += s_loss[i];
        loss_part[blockIdx.y * n_wgs + blockIdx.x] = t;
    }
}

// dL/dW = sigma * sum of the partials + 2 lam W P / ||P||_F, and the SGD update from it; the last block writes
// the loss terms.  64 elements per workgroup of 1024 threads: wave w sums a sixteenth of the partials of
// each, the sixteen meet in LDS in a fixed order.  Bound by reading the partials once (16.8 MB at r = 128 and
// 256 of them, in the caches): four waves with eight loads in flight each took 8 us, and a launch of its own for
// the update 4.6 us on top; 4.9 us now.
__global__ __launch_bounds__(1024) void train_update_kernel(
    float* __restrict__ W, float* __restrict__ v, int r, int n_wgs, float sigma, float lam, float c_sim, float c_bal,
    float lr, float momentum, float weight_decay, const float* __restrict__ dw_part, const float* __restrict__ WP,
    const float* __restrict__ fro_part, const float* __restrict__ colsum, int n_groups,
    const float* __restrict__ bal_part, const float* __restrict__ loss_part, float* __restrict__ grad,
    float* __restrict__ loss) {
    __shared__ float part[16][64];
    __shared__ float s_fro;
    const int tid = threadIdx.x, el = tid & 63, sl = tid >> 6;
    const int count = HATA_D * r;
    const int e = blockIdx.x * 64 + el;  // (count is a multiple of 64; the last block is past it)
    float f = 0.f;
    if (sl == 0) {
        for (int j = el; j < r; j += 64) f += fro_part[j];
        f = sqrtf(wave_sum64(f));
        if (el == 0) s_fro = f;
    }
    if (e < count) {
        float gp[4] = {0.f, 0.f, 0.f, 0.f};
        int wg = (int)((int64_t)sl * n_wgs / 16);
        const int wg_end = (int)((int64_t)(sl + 1) * n_wgs / 16);
        const float* dp = dw_part + e;
        for (; wg < wg_end; wg += 16) {
            float x[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) x[u] = dp[(int64_t)min(wg + u, wg_end - 1) * count];
#pragma unroll
            for (int u = 0; u < 16; ++u) gp[u & 3] += wg + u < wg_end ? x[u] : 0.f;
        }
        part[sl][el] = (gp[0] + gp[1]) + (gp[2] + gp[3]);
        __syncthreads();
        if (sl == 0) {
            float g = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) g += part[i][el];
            g *= sigma;
            if (f > 0.f) g += lam * 2.f * WP[e] / f;
            if (grad) grad[e] = g;
            const float w0 = W[e];
            const float vn = fmaf(momentum, v[e], fmaf(weight_decay, w0, g));
            v[e] = vn;
            W[e] = fmaf(-lr, vn, w0);
        }
        return;
    }
    // similarity: sum of the workgroup partials; balance: squared norm of the column sums
    const int parts = n_wgs * ((r + 127) / 128);
    float ls = 0.f, lb = 0.f;
    for (int i = tid; i < parts; i += 1024) ls += loss_part[i];
    if (colsum)
        for (int j = tid; j < r * n_groups; j += 1024) lb = fmaf(colsum[j], colsum[j], lb);
    else
        for (int i = tid; i < parts; i += 1024) lb += bal_part[i];
    ls = wave_sum64(ls);
    lb = wave_sum64(lb);
    if (el == 0) { part[0][sl] = ls; part[1][sl] = lb; }
    __syncthreads();
    if (tid == 0) {
        ls = lb = 0.f;
        for (int i = 0; i < 16; ++i) { ls += part[0][i]; lb += part[1][i]; }
        loss[0] = c_sim * ls;
        loss[1] = c_bal * lb;
        loss[2] = lam * s_fro;
    }
}

// ---- label builder (App. B.1, steps 3-4) ----------------------------------------------------------
// Rank of a pair = number of pairs with a larger score, or an equal score and a lower index; the first n_pos
// ranks (a tenth of the pairs) get 20 .. 1 in equal steps, the others -1.  Counting every pair against every
// other one costs m^2 compares (571 us at m = 8192), and nine pairs in ten only need to know that they
// are not among the first tenth.  So three launches: the scores, with a coarse histogram of them; from the
// histogram the bin the n_pos-th score lies in -- everything below it is -1, everything from it up goes into a
// candidate list, in any order; ranks by counting inside that list (a hundredth of the compares where the scores
// spread over the bins; m^2 again if they all fall into one).  18 us at m = 8192.
#define LB_BINS 2048
#define LB_COPIES 8     // of the histogram: scores crowd into a few dozen bins, and atomics on one word queue up
#define LB_PASS 16      // scores of a workgroup in one pass

// position of a score in the order of doubles, as an unsigned number (-0 counts as +0; no NaN)
__device__ __forceinline__ unsigned long long score_key(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x + 0.0);
    return (u >> 63) ? ~u : u | (1ull << 63);
}
// its bin, monotone in the score: sign, 64 octaves around 1 (those beyond count as the outermost), 4 mantissa bits
__device__ __forceinline__ int score_bin(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x + 0.0);
    const int step = clampi((int)((u & 0x7fffffffffffffffull) >> 48) - (1023 - 24) * 16, 0, LB_BINS / 2 - 1);
    return (u >> 63) ? LB_BINS / 2 - 1 - step : LB_BINS / 2 + step;
}

// the histogram before the first label call: stream-ordered behind whatever the workspace's memory was used for before
__global__ __launch_bounds__(256) void train_clear_bins_kernel(uint32_t* __restrict__ bins) {
    static_assert(LB_COPIES * LB_BINS % 1024 == 0, "whole workgroups of four words a thread");
    reinterpret_cast<uint4*>(bins)[blockIdx.x * 256 + threadIdx.x] = make_uint4(0, 0, 0, 0);
}

// qk scores of one query against m keys, in fp64 (every product of two bf16 values is exact there): a row
// per 16 lanes, 8 channels per lane; `passes` passes of 16 rows per workgroup.  With several passes the
// workgroup counts in LDS first: fewer device atomics (one copy of the histogram and one pass took 14.7 us
// at m = 8192, nearly all of it queueing on the words of the crowded bins).
__global__ __launch_bounds__(256) void train_scores_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ K,
                                                           int m, int passes, double* __restrict__ scores,
                                                           uint32_t* __restrict__ bins, uint32_t* __restrict__ n_cand) {
    __shared__ uint32_t hist[LB_BINS];
    const int tid = threadIdx.x, sub = tid & 15;
    if (blockIdx.x == 0 && tid == 0) *n_cand = 0;
    if (passes > 1) {
        for (int i = tid; i < LB_BINS; i += 256) hist[i] = 0;
        __syncthreads();
    }
    uint32_t* const mine = bins + (blockIdx.x % LB_COPIES) * LB_BINS;
    const uint4 qv = *reinterpret_cast<const uint4*>(q + sub * 8);
    const uint32_t qw[4] = {qv.x, qv.y, qv.z, qv.w};
    for (int p = 0; p < passes; ++p) {
        const int row = (blockIdx.x * passes + p) * LB_PASS + (tid >> 4);
        double acc = 0.0;
        if (row < m) {
            const uint4 kv = *reinterpret_cast<const uint4*>(K + (int64_t)row * HATA_D + sub * 8);
            const uint32_t kw[4] = {kv.x, kv.y, kv.z, kv.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc = fma((double)bf16_lo(kw[i]), (double)bf16_lo(qw[i]), acc);
                acc = fma((double)bf16_hi(kw[i]), (double)bf16_hi(qw[i]), acc);
            }
        }
        // sum over the 16 lanes of the row, in a fixed order
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 16);
        if (row < m && sub == 0) {
            scores[row] = acc;
            if (acc == acc) atomicAdd(passes > 1 ? &hist[score_bin(acc)] : &mine[score_bin(acc)], 1u);
        }
    }
    if (passes > 1) {
        __syncthreads();
        for (int i = tid; i < LB_BINS; i += 256)
            if (hist[i]) atomicAdd(&mine[i], hist[i]);
    }
}

// label of rank `rank` of n_pos > rank
__device__ __forceinline__ float rank_label(int rank, int n_pos) {
    return (float)(n_pos == 1 ? 20.0 : 20.0 - 19.0 * (double)rank / (double)(n_pos - 1));
}

// 256 pairs per workgroup: the bin that holds the n_pos-th score from the top (every workgroup finds it, the
// histogram is 64 KB), the candidates of its pairs, -1 for the others.  (A NaN score ranks before
// everything and is counted by nobody, as in compares of doubles.)
__global__ __launch_bounds__(256) void train_candidates_kernel(const double* __restrict__ scores, int m, int n_pos,
                                                               const uint32_t* __restrict__ bins,
                                                               uint32_t* __restrict__ n_cand, LabelCand* __restrict__ cand,
                                                               float* __restrict__ s) {
    __shared__ uint32_t scan4[4];
    __shared__ int s_bin;
    __shared__ uint32_t s_base;
    const int tid = threadIdx.x;
    const int i = blockIdx.x * 256 + tid;
    const double x = i < m ? scores[i] : 0.0;
    // thread t owns the eight bins 8 t' .. 8 t' + 7, t' = 255 - t: the scan runs from the top
    const int b0 = (255 - tid) * (LB_BINS / 256);
    uint4 lo[LB_COPIES], hi[LB_COPIES];
#pragma unroll
    for (int c = 0; c < LB_COPIES; ++c) {
        lo[c] = *reinterpret_cast<const uint4*>(bins + c * LB_BINS + b0);
        hi[c] = *reinterpret_cast<const uint4*>(bins + c * LB_BINS + b0 + 4);
    }
    uint32_t h[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < LB_COPIES; ++c) {
        h[0] += hi[c].w; h[1] += hi[c].z; h[2] += hi[c].y; h[3] += hi[c].x;
        h[4] += lo[c].w; h[5] += lo[c].z; h[6] += lo[c].y; h[7] += lo[c].x;
    }
    uint32_t loc = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) loc += h[j];
    if (tid == 0) s_bin = 0;  // (fewer scores than n_pos: NaNs)
    uint32_t total;
    uint32_t run = block_excl_scan_256(loc, scan4, &total);
    if (run < (uint32_t)n_pos && run + loc >= (uint32_t)n_pos) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (run < (uint32_t)n_pos && run + h[j] >= (uint32_t)n_pos) s_bin = b0 + 7 - j;
            run += h[j];
        }
    }
    __syncthreads();
    const bool nan = !(x == x);
    const bool take = i < m && !nan && score_bin(x) >= s_bin;
    if (i < m && !take) s[i] = nan ? rank_label(0, n_pos) : -1.f;
    const uint32_t before = block_excl_scan_256(take ? 1u : 0u, scan4, &total);
    if (total == 0) return;
    if (tid == 0) s_base = atomicAdd(n_cand, total);
    __syncthreads();
    if (take) {
        LabelCand c;
        c.key = score_key(x); c.row = (uint32_t)i; c.pad = 0;
        cand[s_base + before] = c;
    }
}

// ranks inside the candidate list: 64 candidates per workgroup and turn, each counted by sixteen waves over a
// sixteenth of the list; the histogram is cleared for the next call
__global__ __launch_bounds__(1024) void train_labels_kernel(const LabelCand* __restrict__ cand, const uint32_t* __restrict__ n_cand,
                                                            int n_pos, uint32_t* __restrict__ bins, float* __restrict__ s) {
    __shared__ int s_rank[16][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x == gridDim.x - 1)
        for (int i = tid; i < LB_COPIES * LB_BINS; i += 1024) bins[i] = 0;
    const int nc = (int)*n_cand;
    for (int c0 = blockIdx.x * 64; c0 < nc; c0 += gridDim.x * 64) {
        const LabelCand me = cand[min(c0 + lane, nc - 1)];
        int rank = 0;
        for (int j = wave * 64; j < nc; j += 16 * 64) {
            // 64 entries, one per lane, handed round as scalars; key 0 (behind every score) past the end
            const LabelCand o = cand[min(j + lane, nc - 1)];
            const bool live = j + lane < nc;
            const int klo = live ? (int)(uint32_t)o.key : 0, khi = live ? (int)(uint32_t)(o.key >> 32) : 0;
#pragma unroll
            for (int t = 0; t < 64; ++t) {
                const unsigned long long key = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane(khi, t) << 32) |
                                               (uint32_t)__builtin_amdgcn_readlane(klo, t);
                const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)o.row, t);
                rank += (key > me.key || (key == me.key && row < me.row)) ? 1 : 0;
            }
        }
        s_rank[wave][lane] = rank;
        __syncthreads();
        if (wave == 0 && c0 + lane < nc) {
            rank = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) rank += s_rank[i][lane];
            s[me.row] = rank < n_pos ? rank_label(rank, n_pos) : -1.f;
        }
        __syncthreads();
    }
}

}  // namespace hata

namespace {
constexpr size_t kAlignT = 256;
inline size_t align_up_t(size_t x) { return (x + kAlignT - 1) / kAlignT * kAlignT; }
struct TrainPlan { int n_wgs_max; size_t off_colsum, off_cs, off_bal, off_dw, off_loss, off_P, off_fro, off_WP, off_planes, off_scores, off_bins, off_ncand, off_cand, total; };
int make_train_plan(const hata_train_config* f, TrainPlan* p) {
    if (!f) return HATA_EINVAL;
    if (f->n_max < 1) return HATA_EINVAL;
    if (f->d != 128) return HATA_EUNSUPPORTED;
    if (f->r != 32 && f->r != 64 && f->r != 128 && f->r != 256) return HATA_EUNSUPPORTED;
    p->n_wgs_max = (f->n_max + TR_ROWS - 1) / TR_ROWS;
    if (p->n_wgs_max > 65535) return HATA_EUNSUPPORTED;
    size_t o = 0;
    p->off_colsum = o; o = align_up_t(o + (size_t)p->n_wgs_max * f->r * 4);
    p->off_cs = o;     o = align_up_t(o + (size_t)p->n_wgs_max * f->r * 4);
    p->off_dw = o;     o = align_up_t(o + (size_t)p->n_wgs_max * f->d * f->r * 4);
    p->off_loss = o;   o = align_up_t(o + (size_t)p->n_wgs_max * 2 * 4);
    p->off_P = o;      o = align_up_t(o + (size_t)f->r * f->r * 4);
    p->off_fro = o;    o = align_up_t(o + (size_t)f->r * 4);
    p->off_WP = o;     o = align_up_t(o + (size_t)f->d * f->r * 4);
    p->off_planes = o; o = align_up_t(o + (size_t)f->r / 32 * 3 * 8 * 64 * 16);
    p->off_bal = o;    o = align_up_t(o + (size_t)p->n_wgs_max * 2 * 4);
    p->off_scores = o; o = align_up_t(o + (size_t)f->n_max * 8);
    p->off_bins = o;   o = align_up_t(o + (size_t)LB_COPIES * LB_BINS * 4);
    p->off_ncand = o;  o = align_up_t(o + 4);
    p->off_cand = o;   o = align_up_t(o + (size_t)f->n_max * sizeof(LabelCand));
    p->total = o;
    return HATA_OK;
}
}  // namespace

extern "C" {

int hata_train_workspace_bytes(const hata_train_config* cfg, size_t* out) {
    if (!out) return HATA_EINVAL;
    TrainPlan p;
    const int rc = make_train_plan(cfg, &p);
    if (rc != HATA_OK) return rc;
    *out = p.total;
    return HATA_OK;
}

int hata_train_create(hata_train_ctx** ctx_out, const hata_train_config* cfg, void* workspace,
                      size_t workspace_bytes) {
    if (!ctx_out) return HATA_EINVAL;
    *ctx_out = nullptr;
    TrainPlan p;
    const int rc = make_train_plan(cfg, &p);
    if (rc != HATA_OK) return rc;
    if (!workspace || ((uintptr_t)workspace % kAlignT) != 0 || workspace_bytes < p.total) return HATA_EWORKSPACE;
    hata_train_ctx* c = new (std::nothrow) hata_train_ctx;
    if (!c) return HATA_EINVAL;
    c->cfg = *cfg;
    c->n_wgs_max = p.n_wgs_max;
    char* w = (char*)workspace;
    c->colsum_part = (float*)(w + p.off_colsum);
    c->colsum = (float*)(w + p.off_cs);
    c->dw_part = (float*)(w + p.off_dw);
    c->loss_part = (float*)(w + p.off_loss);
    c->P = (float*)(w + p.off_P);
    c->fro_part = (float*)(w + p.off_fro);
    c->WP = (float*)(w + p.off_WP);
    c->planes = (uint4*)(w + p.off_planes);
    c->bal_part = (float*)(w + p.off_bal);
    c->scores = (double*)(w + p.off_scores);
    c->bins = (uint32_t*)(w + p.off_bins);
    c->n_cand = (uint32_t*)(w + p.off_ncand);
    c->cand = (LabelCand*)(w + p.off_cand);
    c->bins_clear = 0;
    *ctx_out = c;
    return HATA_OK;
}

int hata_train_destroy(hata_train_ctx* ctx) {
    delete ctx;
    return HATA_OK;
}

int hata_train_step(hata_train_ctx* ctx, const void* Q, const void* K, const float* s, int32_t n,
                    const int32_t* block_query, int32_t n_queries, float* W, float* v,
                    const hata_train_hparams* hp, float* grad, float* loss, void* stream) {
    if (!ctx || !Q || !K || !s || !W || !v || !hp) return HATA_EINVAL;
    if (n < 1 || n > ctx->cfg.n_max) return HATA_EINVAL;
    if (!block_query) n_queries = 1;
    if (n_queries < 1 || n_queries > (n + TR_ROWS - 1) / TR_ROWS || ((uintptr_t)block_query % 4)) return HATA_EINVAL;
    if (((uintptr_t)Q % 16) || ((uintptr_t)K % 16) || ((uintptr_t)W % 16) || ((uintptr_t)v % 4) || ((uintptr_t)s % 4))
        return HATA_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    const int r = ctx->cfg.r;
    const int n_wgs = (n + TR_ROWS - 1) / TR_ROWS;
    const float c_sim = hp->eps * hp->scale_sim, c_bal = hp->eta * hp->scale_bal;
    const uint16_t* q = (const uint16_t*)Q;
    const uint16_t* k = (const uint16_t*)K;
    const bool few = n_wgs <= TR_FEW_WGS;
    const float* colsum = few ? nullptr : ctx->colsum;
#define HATA_TRAIN_LAUNCH(RR)                                                                          \
    do {                                                                                               \
        using S = hata::TrainShape<RR>;                                                                \
        hipLaunchKernelGGL((hata::train_colsum_kernel<RR>), dim3(n_wgs + 8 + S::COLS, RR / S::COLS),   \
                           dim3(S::THREADS), 0, st, k, W, n, n_wgs, hp->sigma, ctx->colsum_part,       \
                           ctx->P, ctx->fro_part, ctx->planes);                                        \
        if (!few)                                                                                      \
            hipLaunchKernelGGL(hata::train_colreduce_kernel, dim3(RR, n_queries), dim3(256), 0, st,    \
                               ctx->colsum_part, RR, n_wgs, block_query, n_queries, ctx->colsum);      \
        hipLaunchKernelGGL((hata::train_grad_kernel<RR>), dim3(n_wgs + HATA_D, RR / S::COLS),          \
                           dim3(S::THREADS), 0, st, q, k, s, W, ctx->planes, n, n_wgs, hp->sigma,      \
                           c_sim, c_bal, colsum, ctx->colsum_part, block_query, n_queries, ctx->P,     \
                           ctx->dw_part, ctx->loss_part, ctx->bal_part, ctx->WP);                      \
    } while (0)
    switch (r) {
        case 32: HATA_TRAIN_LAUNCH(32); break;
        case 64: HATA_TRAIN_LAUNCH(64); break;
        case 128: HATA_TRAIN_LAUNCH(128); break;
        default: HATA_TRAIN_LAUNCH(256); break;
    }
#undef HATA_TRAIN_LAUNCH
    hipLaunchKernelGGL(hata::train_update_kernel, dim3(HATA_D * r / 64 + (loss ? 1 : 0)), dim3(1024), 0, st, W, v, r, n_wgs,
                       hp->sigma, hp->lam, c_sim, c_bal, hp->lr, hp->momentum, hp->weight_decay, ctx->dw_part, ctx->WP,
                       ctx->fro_part, colsum, n_queries, ctx->bal_part, ctx->loss_part, grad, loss);
    return hipGetLastError() == hipSuccess ? HATA_OK : HATA_EHIP;
}

int hata_train_make_labels(hata_train_ctx* ctx, const void* q, const void* K, int32_t m, float* s,
                           void* stream) {
    if (!ctx || !q || !K || !s) return HATA_EINVAL;
    if (m < 1 || m > ctx->cfg.n_max) return HATA_EINVAL;
    if (((uintptr_t)q % 16) || ((uintptr_t)K % 16) || ((uintptr_t)s % 4)) return HATA_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    int n_pos = m / 10;
    if (n_pos < 1) n_pos = 1;
    const int passes = m <= 16384 ? 1 : m / 8192 < 32 ? m / 8192 : 32;
    // Nothing is written to the workspace before the first call, which clears the histogram on its own stream; every call
    // leaves it clear (train_labels_kernel).  A clear that is only recorded into a graph has not run yet, so it
    // does not count: the graph clears at each replay and the next call still does.
    bool cleared = ctx->bins_clear != 0;
    if (!cleared) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusActive;
        const hipError_t e = hipStreamIsCapturing(st, &capture);
        if (e != hipSuccess) (void)hipGetLastError();
        cleared = e == hipSuccess && capture == hipStreamCaptureStatusNone;
        hipLaunchKernelGGL(hata::train_clear_bins_kernel, dim3(LB_COPIES * LB_BINS / 1024), dim3(256), 0, st, ctx->bins);
    }
    hipLaunchKernelGGL(hata::train_scores_kernel, dim3((m + LB_PASS * passes - 1) / (LB_PASS * passes)), dim3(256), 0, st,
                       (const uint16_t*)q, (const uint16_t*)K, m, passes, ctx->scores, ctx->bins, ctx->n_cand);
    hipLaunchKernelGGL(hata::train_candidates_kernel, dim3((m + 255) / 256), dim3(256), 0, st, ctx->scores, m, n_pos,
                       ctx->bins, ctx->n_cand, ctx->cand, s);
    // enough workgroups for twice the expected list (they take more turns if it is longer)
    hipLaunchKernelGGL(hata::train_labels_kernel, dim3(n_pos / 32 + 2), dim3(1024), 0, st, ctx->cand, ctx->n_cand, n_pos,
                       ctx->bins, s);
    const bool ok = hipGetLastError() == hipSuccess;
    ctx->bins_clear = ok && cleared;  // (after a call that failed half-way the next one clears again)
    return ok ? HATA_OK : HATA_EHIP;
}

}  // extern "C"
