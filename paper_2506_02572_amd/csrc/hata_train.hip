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
// Launches of a step (two, three where the column sums have a launch of their own):
//   1. train_grad_kernel, train_grad_runs_kernel (batches of more than a round of workgroups)
//                            The balance term couples every row to the sum of h(k) over its query, but only through
//                            a factor per hash column: dL/dz_k = (c_j - a_n) e_n with e = 1 - h(k)^2, so
//                            K^T dZ_k = c_j K^T E - K^T (A E), and the two contractions need no sums.
//                            So one pass over the triplets: forward of k and q, K^T E and K^T (A E) with the MFMA
//                            result registers as the B operand (the contraction index -- the row -- may be
//                            enumerated in any order, so the 32x32 result layout is used as it stands;
//                            only X is read transposed, from the LDS tile it was staged in) -> partial sums of both
//                            and column sums of h(k) per workgroup;
//                            on the way: W W^T in fp64, half a row per workgroup, and a copy of W
//      (train_colreduce_kernel adds the column sums up per query where the next launch's workgroups would have too
//      many to do so themselves)
//   2. train_update_kernel   dL/dW = sigma sum partials + 2 lam W P / ||P||_F with W P = (W W^T) W - W, the loss
//                            terms, weight decay, momentum, step
// At r = 128 and 32768 triplets of four queries a step takes 27 us (29 with a workgroup per pair of blocks), at 122880 triplets 64 (86).
#include <new>
#include <type_traits>

#include "hata_device.h"
#include "../../include/hata_train.h"

struct LabelCand { unsigned long long key; uint32_t row, pad; };

struct hata_train_ctx {
    hata_train_config cfg;
    int n_wgs_max;
    float* colsum_part;  // [n_wgs_max, r]
    float* colsum;       // [queries (<= n_wgs_max), r]  sum of h(k_n) over the triplets of a query
    float* dw_part;      // [pairs of blocks, 3, d, r]  K^T E, the rest of X^T dZ, K^T E of the second block if its query is another; a run's: in its last pair's place, the K^T E of a query that ends sooner in its own last pair's
    float* loss_part;    // [column groups, pairs of blocks]
    double* gram;        // [d, d]  W W^T
    double* fro_part;    // [2 d]  what its pieces add to ||W^T W - I||_F^2 - r
    float* W_old;        // [d, r]  the weights the gradient was taken at (the update overwrites W as it goes)
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
#define TR_ROWS 128   // triplets per block: those of one query
#define TR_PAIR 256   // triplets per workgroup: two blocks (one LDS stage)
#define TR_ONE_ROUND 256  // workgroups of the gradient launch that run side by side, one per CU
#define TR_FEW_WGS 512    // up to so many blocks and queries every workgroup of the update adds the column sums up itself
#define TR_FEW_QUERIES 32
#define TR_UPDATE_WAVES 8  // waves of an update workgroup
#define TR_PITCH 136  // LDS row pitch in bf16 elements (272 B: conflict-free 16-B and transposed reads)
#define TR_KEPT 4      // stages of a workgroup whose column sums are kept until they are written

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

// How a workgroup's eight waves share its TR_PAIR rows and COLS = 32 or 64 hash columns: a wave owns 32 columns and
// 1 / RG of the rows.  Half the columns and twice the rows of a 128-column tile cost as many partial sums, two contractions
// instead of one included.
template <int COLS_>
struct TrainShape {
    static constexpr int COLS = COLS_;
    static constexpr int CG = COLS / 32;
    static constexpr int WAVES = 8, THREADS = WAVES * 64;
    static constexpr int RG = WAVES / CG;            // row groups
    static constexpr int HB = RG / 2;                // of a block
    static constexpr int TILES = TR_PAIR / 32 / RG;  // 32-row tiles of a wave
    static constexpr int COL_ROWS = WAVES > THREADS / COLS ? WAVES : THREADS / COLS;  // rows of per-column sums: for any split over waves or threads (the row groups have one each)
};

// rows [row0, row0 + TR_PAIR) of X [n, 128] (row0 < n): fetched into registers -- past n the last row, so that no load
// is behind a branch -- and, once they are zeroed there, put into an LDS tile
template <int THREADS>
struct StagedRows {
    static constexpr int NV = TR_PAIR * 16 / THREADS;
    uint4 v[NV];
    __device__ __forceinline__ void fetch(const uint16_t* __restrict__ X, int row0, int n) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = threadIdx.x + j * THREADS, row = min(row0 + (i >> 4), n - 1), sub = i & 15;
            v[j] = *reinterpret_cast<const uint4*>(X + (int64_t)row * HATA_D + sub * 8);
        }
    }
    __device__ __forceinline__ void zero_past(int row0, int n) {
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (row0 + (int)((threadIdx.x + j * THREADS) >> 4) >= n) v[j] = make_uint4(0, 0, 0, 0);
    }
    __device__ __forceinline__ void put(uint16_t* tile) const {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = threadIdx.x + j * THREADS, row = i >> 4, sub = i & 15;
            *reinterpret_cast<uint4*>(&tile[row * TR_PITCH + sub * 8]) = v[j];
        }
    }
};

// Z tiles t0 .. (32 rows x the wave's 32 columns each) = X_tile . W: result register ri of lane (m, half)
// holds row 8 (ri / 4) + 4 half + ri % 4 of the tile, column 32 w + m
template <int TILES>
__device__ __forceinline__ void project_tiles(const uint16_t* tile, int t0, int m, int half, const tr_bf16x8_t (&wfrag)[3][8],
                                              tr_f32x16_t (&z)[TILES]) {
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) z[t][i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const tr_bf16x8_t x = *reinterpret_cast<const tr_bf16x8_t*>(&tile[((t0 + t) * 32 + m) * TR_PITCH + kk * 16 + 8 * half]);
#pragma unroll
            for (int p = 0; p < 3; ++p) z[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, wfrag[p][kk], z[t], 0, 0, 0);
        }
    }
}

// the query a block of TR_ROWS triplets belongs to (no names: everything is query 0; a name outside
// [0, n_groups) counts as the nearest valid one, so no access leaves the arrays)
__device__ __forceinline__ int block_query(const int32_t* __restrict__ block_group, int wg, int n_groups) {
    return block_group ? clampi(block_group[wg], 0, n_groups - 1) : 0;
}

// The blocks' column sums added up per query: a workgroup per (64 hash columns, query), a wave a sixteenth of the blocks.  It
// looks up 64 blocks' queries at a time, a lane each, and reads whole rows of its own query's blocks, so that many queries
// are many short workgroups (with a workgroup per column and query, a thread per block, a step of 960 blocks of as many queries,
// r = 128, took 224 us, 158 so, 122 with the loss term's sums read sixteen at a time too).
#define TR_REDUCE_WAVES 16
__global__ __launch_bounds__(TR_REDUCE_WAVES * 64) void train_colreduce_kernel(const float* __restrict__ colsum_part, int r,
                                                                               int n_blocks, const int32_t* __restrict__ block_group,
                                                                               int n_groups, float* __restrict__ colsum) {
    __shared__ float part[TR_REDUCE_WAVES][64];
    const int tid = threadIdx.x, el = tid & 63, sl = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = blockIdx.y, j = min((int)blockIdx.x * 64 + el, r - 1);
    float acc = 0.f;
    for (int b = 64 * sl; b < n_blocks; b += 64 * TR_REDUCE_WAVES) {
        const int id = block_query(block_group, min(b + el, n_blocks - 1), n_groups);
        unsigned long long own = __builtin_amdgcn_ballot_w64(id == q && b + el < n_blocks);
        if (own == 0) continue;
        const float* const rows = colsum_part + (int64_t)b * r + j;
        if (__popcll(own) > 8) {
            const int last = 63 - __builtin_clzll(own);
#pragma unroll
            for (int h = 0; h < 64; h += 32) {
                float x[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) x[u] = rows[(int64_t)min(h + u, last) * r];
#pragma unroll
                for (int u = 0; u < 32; ++u) acc += (own >> (h + u)) & 1 ? x[u] : 0.f;
            }
        } else {
            float x[8];
            int at = 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool more = own != 0;
                if (more) at = __builtin_ctzll(own);
                own &= own - 1;
                const float y = rows[(int64_t)at * r];
                x[u] = more ? y : 0.f;
            }
            acc += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
        }
    }
    part[sl][el] = acc;
    __syncthreads();
    if (sl == 0) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < TR_REDUCE_WAVES; ++i) t += part[i][el];
        if ((int)blockIdx.x * 64 + el < r) colsum[(int64_t)q * r + j] = t;
    }
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

// eight consecutive values of a result (registers 8 ks .. 8 ks + 7), split for the B operand
__device__ __forceinline__ void split_operand(const tr_f32x16_t& v, int ks, tr_bf16x8_t (&b)[3]) {
    uint32_t pz[3][4];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) split3_pair(v[8 * ks + 2 * e2], v[8 * ks + 2 * e2 + 1], pz[0][e2], pz[1][e2], pz[2][e2]);
#pragma unroll
    for (int p = 0; p < 3; ++p) b[p] = __builtin_bit_cast(tr_bf16x8_t, make_uint4(pz[p][0], pz[p][1], pz[p][2], pz[p][3]));
}

// sum over a wave's lanes, in fp64
__device__ __forceinline__ double wave_sum64_f64(double x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

// Half rows of W W^T and rows of a copy of W, a piece of each per workgroup of 512 threads: what a thread needs of
// it, requested ahead of its use
template <int R>
struct GramPiece {
    static constexpr int PIECES = 2 * HATA_D;  // piece c: row c / 2, channels 64 (c % 2) ...
    static constexpr int NV = R / 32;          // eight threads per element
    float4 a[NV], b[NV];
    float w;
    __device__ __forceinline__ void fetch(const float* __restrict__ W, int c) {
        const int tid = threadIdx.x, ch = (c & 1) * 64 + (tid >> 3), part = tid & 7;
        const float4* ra = reinterpret_cast<const float4*>(W + (int64_t)ch * R) + part;
        const float4* rb = reinterpret_cast<const float4*>(W + (int64_t)(c >> 1) * R) + part;
#pragma unroll
        for (int i = 0; i < NV; ++i) { a[i] = ra[8 * i]; b[i] = rb[8 * i]; }
        w = (c & 1) == 0 && tid < R ? W[(int64_t)(c >> 1) * R + tid] : 0.f;
    }
    // returns this wave's part of ||W W^T||^2 - 2 tr(W W^T)  (||W^T W - I||^2 = that + r)
    __device__ __forceinline__ double finish(int c, double* __restrict__ gram, float* __restrict__ W_old) const {
        const int tid = threadIdx.x, row = c >> 1, ch = (c & 1) * 64 + (tid >> 3);
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            acc = fma((double)a[i].x, (double)b[i].x, acc);
            acc = fma((double)a[i].y, (double)b[i].y, acc);
            acc = fma((double)a[i].z, (double)b[i].z, acc);
            acc = fma((double)a[i].w, (double)b[i].w, acc);
        }
        acc += __shfl_xor(acc, 1, 64);
        acc += __shfl_xor(acc, 2, 64);
        acc += __shfl_xor(acc, 4, 64);
        if ((tid & 7) == 0) gram[row * HATA_D + ch] = acc;
        if ((c & 1) == 0 && tid < R) W_old[(int64_t)row * R + tid] = w;
        double f = acc * acc - (ch == row ? 2.0 * acc : 0.0);
        f += __shfl_xor(f, 8, 64);
        f += __shfl_xor(f, 16, 64);
        return f + __shfl_xor(f, 32, 64);
    }
};

// The same without the registers of requests made ahead: four loads of either row at a time
template <int R>
__device__ __forceinline__ double gram_piece(const float* __restrict__ W, int c, int tid, double* __restrict__ gram, float* __restrict__ W_old) {
    constexpr int NV = R / 32 < 4 ? R / 32 : 4;  // eight threads per element, NV loads of either row in flight (registers)
    const int row = c >> 1, ch = (c & 1) * 64 + (tid >> 3), part = tid & 7;
    const float4* ra = reinterpret_cast<const float4*>(W + ch * R) + part;
    const float4* rb = reinterpret_cast<const float4*>(W + row * R) + part;
    const bool copies = (c & 1) == 0 && tid < R;
    const float w = copies ? W[row * R + tid] : 0.f;
    double acc = 0.0;
#pragma clang loop unroll(disable)
    for (int i0 = 0; i0 < R / 32; i0 += NV) {
        float4 a[NV], b[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) { a[i] = ra[8 * (i0 + i)]; b[i] = rb[8 * (i0 + i)]; }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            acc = fma((double)a[i].x, (double)b[i].x, acc);
            acc = fma((double)a[i].y, (double)b[i].y, acc);
            acc = fma((double)a[i].z, (double)b[i].z, acc);
            acc = fma((double)a[i].w, (double)b[i].w, acc);
        }
    }
    acc += __shfl_xor(acc, 1, 64);
    acc += __shfl_xor(acc, 2, 64);
    acc += __shfl_xor(acc, 4, 64);
    if (part == 0) gram[row * HATA_D + ch] = acc;
    if (copies) W_old[row * R + tid] = w;
    double f = acc * acc - (ch == row ? 2.0 * acc : 0.0);
    f += __shfl_xor(f, 8, 64);
    f += __shfl_xor(f, 16, 64);
    return f + __shfl_xor(f, 32, 64);
}

// grid = (pairs of blocks of TR_ROWS triplets, groups of COLS hash columns).
//
// A block whose rows hold one query vector -- those of a sampled query against its keys do; rows of zeros with label 0
// fill such a block up -- needs that vector projected once, and its part of Q^T dZ_q is that vector times a sum over
// the rows.  Whether it does is looked up in the rows themselves; a workgroup with any other row takes the general way.
//
// What bounds it: the way of a workgroup, one per CU and in step throughout, from what it reads (4 us to the first product)
// over the matrix instructions (of a wave 48 for the projection of its keys, 24 for the query, 96 for the two contractions; the
// general way has 72 more, and stages the keys twice) with the exponentials and the splits, to its sums.  So the reads are
// requested together, behind no branch, and small batches have workgroups of 32 columns, half the way.  Kernel time at r = 128, us,
// one query vector a block / others: one block 11.0 / 13.6 (64 columns 14.5 / 20.1), 256 blocks 20.0 / 25.4 (21.1 / 26.9 with
// the reads one after the other).  Larger batches, unless their queries are short, take train_grad_runs_kernel.  With a launch for the column sums
// in front and both tiles side by side the general way was ahead in the smallest batches of r = 32 (one block a step 16.7, 19.1 so).
template <int R, int COLS>
__global__ __launch_bounds__(TrainShape<COLS>::THREADS) void train_grad_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const float* __restrict__ s, const float* __restrict__ W,
    int n, int n_blocks, float sigma, float c_sim, const int32_t* __restrict__ block_group, int n_groups,
    float* __restrict__ dw_part, float* __restrict__ colsum_part, float* __restrict__ loss_part, double* __restrict__ gram,
    double* __restrict__ fro_part, float* __restrict__ W_old) {
    using S = TrainShape<COLS>;
    constexpr int THREADS = S::THREADS, WAVES = S::WAVES, T = S::TILES;
    __shared__ __attribute__((aligned(16))) uint16_t tile[TR_PAIR * TR_PITCH];
    __shared__ __attribute__((aligned(16))) uint16_t s_q[2][HATA_D];  // first query row of each block
    // operand fragments: the planes of the weights [CG][3][8], later those of a round's values [CG][RG][6]
    __shared__ __attribute__((aligned(16))) uint4 s_frag[48][64];
    static_assert(S::CG * 3 * 8 <= 48 && S::CG * S::RG * 6 <= 48, "fragments");
    __shared__ float s_lab[TR_PAIR];
    __shared__ float s_col[S::COL_ROWS][COLS];  // per hash column: sums of h(k_n) over a row group
    __shared__ float s_dq[S::RG][COLS];  // sums of dZ_q
    __shared__ float s_loss[WAVES];
    __shared__ double s_red[WAVES];
    __shared__ int s_mixed;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = (tid >> 6) % S::CG, rg = (tid >> 6) / S::CG;
    const int m = lane & 31, half = lane >> 5;
    const int row0 = blockIdx.x * TR_PAIR, blk = rg / S::HB;
    const int col = blockIdx.y * COLS + w * 32 + m;
    const int wg = blockIdx.y * gridDim.x + blockIdx.x, first = 2 * blockIdx.x;
    GramPiece<R> piece;
    if (first >= n_blocks) {  // (small batches have workgroups for the pieces alone)
        if (wg < GramPiece<R>::PIECES) {
            piece.fetch(W, wg);
            const double f = piece.finish(wg, gram, W_old);
            if (lane == 0) s_red[tid >> 6] = f;
            __syncthreads();
            if (tid == 0) {
                double t = 0.0;
                for (int i = 0; i < WAVES; ++i) t += s_red[i];
                fro_part[wg] = t;
            }
        }
        return;
    }
    // everything the workgroup reads is requested before any of it is waited for; what it needs last, last
    StagedRows<THREADS> xk, xq;
    xk.fetch(K, row0, n);
    // the planes of the column group's weights, a share of the channel steps by each of its row groups
    constexpr int KS = 8 / S::RG;
    float wv[KS][8];
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) wv[k][e] = W[(int64_t)((rg * KS + k) * 16 + 8 * half + e) * R + col];
    xq.fetch(Q, row0, n);
    const int lab_row = row0 + (tid & (TR_PAIR - 1));
    const float lab = s[min(lab_row, n - 1)];
    if (wg < GramPiece<R>::PIECES) piece.fetch(W, wg);
    const bool one_query = first + 1 >= n_blocks || block_query(block_group, first, n_groups) == block_query(block_group, first + 1, n_groups);
    if (tid == 0) s_mixed = 0;
    xk.zero_past(row0, n);
    xk.put(tile);
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        uint32_t f[3][4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) split3_pair(wv[k][2 * e2], wv[k][2 * e2 + 1], f[0][e2], f[1][e2], f[2][e2]);
#pragma unroll
        for (int p = 0; p < 3; ++p) s_frag[(w * 3 + p) * 8 + rg * KS + k][lane] = make_uint4(f[p][0], f[p][1], f[p][2], f[p][3]);
    }
    if (tid < TR_PAIR) s_lab[tid] = lab_row < n ? lab : 0.f;
    // thread: piece tid % 16 of rows tid / 16 + 32 j
    xq.zero_past(row0, n);
    if (tid < 16) {
        *reinterpret_cast<uint4*>(&s_q[0][tid * 8]) = xq.v[0];
        *reinterpret_cast<uint4*>(&s_q[1][tid * 8]) = xq.v[TR_ROWS * 16 / THREADS];
    }
    {
        double fro = 0.0;
        if (wg < GramPiece<R>::PIECES) fro = piece.finish(wg, gram, W_old);
        if (lane == 0) s_red[tid >> 6] = fro;
    }
    __syncthreads();
    {
        uint32_t stray = 0;  // (no branches: every read is in flight at once)
        uint4 f[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) f[b] = *reinterpret_cast<const uint4*>(&s_q[b][(tid & 15) * 8]);
#pragma unroll
        for (int j = 0; j < StagedRows<THREADS>::NV; ++j) {
            const int row = (tid >> 4) + j * (THREADS / 16), b = j / (StagedRows<THREADS>::NV / 2);
            const uint4 x = xq.v[j];
            const uint32_t differs = (x.x ^ f[b].x) | (x.y ^ f[b].y) | (x.z ^ f[b].z) | (x.w ^ f[b].w);
            const uint32_t counts = x.x | x.y | x.z | x.w | (__float_as_uint(s_lab[row]) << 1);  // (a label of -0 is 0)
            stray |= counts != 0u ? differs : 0u;
        }
        if (stray) s_mixed = 1;
    }
    tr_bf16x8_t wfrag[3][8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
#pragma unroll
        for (int p = 0; p < 3; ++p) wfrag[p][kk] = __builtin_bit_cast(tr_bf16x8_t, s_frag[(w * 3 + p) * 8 + kk][lane]);
    const float nsl = -sigma * TR_LOG2E;
    const int t0 = rg * T;
    tr_f32x16_t zk[T];  // then h(k)
    project_tiles<T>(tile, t0, m, half, wfrag, zk);
    __syncthreads();
    const bool mixed = s_mixed != 0;
    float lsim = 0.f, cs = 0.f, ssum = 0.f;  // similarity, sum of h(k), sum of s (h(q) - h(k))
    tr_f32x16_t zq[T];  // then h(q)
    float hq0 = 0.f;
    if (mixed) {
        xq.put(tile);
        __syncthreads();
        project_tiles<T>(tile, t0, m, half, wfrag, zq);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) zq[t][i] = relaxed_sign(zq[t][i], nsl);
    } else {
        tr_f32x16_t z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const tr_bf16x8_t x = *reinterpret_cast<const tr_bf16x8_t*>(&s_q[blk][kk * 16 + 8 * half]);
#pragma unroll
            for (int p = 0; p < 3; ++p) z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, wfrag[p][kk], z, 0, 0, 0);
        }
        hq0 = relaxed_sign(z[0], nsl);
    }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float hk = relaxed_sign(zk[t][i], nsl);
            zk[t][i] = hk;
            cs += hk;  // (rows past n are zero: h = 0)
        }
    // Every wave has the values of its rows, and gets the sums over all of them (RG = 8: over one block's) for 32
    // channels: a round hands 16 rows of each row group round through LDS, split into planes.  (With sums of its own rows over
    // all channels instead, a wave held 128 of them, its products waited for one operand at a time, and the
    // sums had to be added up through LDS: 14 us of that against 8.)
    // accumulators: channel 32 ct + 8 (ri / 4) + 4 half + ri % 4, this lane's column
    const int ct = rg & 3;
    constexpr int G0 = S::RG == 8 ? 4 : S::RG;  // row groups a wave adds up
    const int g0 = S::RG == 8 ? (rg & 4) : 0;
    tr_f32x16_t ke[2], dw;  // K^T E, by block (RG = 8: the wave's block in both places);  Q^T dZ_q - K^T (A E)
#pragma unroll
    for (int i = 0; i < 16; ++i) ke[0][i] = ke[1][i] = dw[i] = 0.f;
    // where this lane reads of a 4-row x 16-channel piece of a tile (lds_read_transposed), for row group
    // 4 half and channel group 16 (m / 16)
    const uint16_t* const tr = tile + (4 * half + (lane & 15) / 4) * TR_PITCH + 16 * (m >> 4) + 4 * (lane & 3);
    // X: 16 rows (slot (half, j) of the operand <-> row 8 (j / 4) + 4 half + j % 4), 32 channels
    auto rows_transposed = [&](int t, int ks) {
        const uint16_t* p = tr + (t * 32 + 16 * ks) * TR_PITCH + 32 * ct;
        const uint2 lo = lds_read_transposed(p), hi = lds_read_transposed(p + 8 * TR_PITCH);
        return __builtin_bit_cast(tr_bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
    };
    tr_bf16x8_t b[6];  // planes of the next round's values
    auto hand_round = [&]() {
#pragma unroll
        for (int p = 0; p < 6; ++p) s_frag[(w * S::RG + rg) * 6 + p][lane] = __builtin_bit_cast(uint4, b[p]);
        __syncthreads();
    };
    auto handed = [&](int g, int p) { return __builtin_bit_cast(tr_bf16x8_t, s_frag[(w * S::RG + g0 + g) * 6 + p][lane]); };
    // 16 rows' E and -A E
    auto prepare_keys = [&](int round, auto one_vector) {
        const int t = round / 2, ks = round % 2;
        tr_f32x16_t e, ae;
#pragma unroll
        for (int i = 8 * ks; i < 8 * ks + 8; ++i) {
            // (half of dL/dh: h' = (1 - h^2) / 2)
            float hq = hq0;
            if constexpr (!decltype(one_vector)::value) hq = zq[t][i];
            const float hk = zk[t][i], diff = hq - hk, sd = s_lab[(t0 + t) * 32 + 8 * (i / 4) + 4 * half + (i % 4)] * diff;
            e[i] = fmaf(-hk, hk, 1.f);
            ae[i] = -c_sim * sd * e[i];
            lsim = fmaf(sd, diff, lsim);
            ssum += sd;
        }
        tr_bf16x8_t be[3], ba[3];
        split_operand(e, ks, be);
        split_operand(ae, ks, ba);
#pragma unroll
        for (int p = 0; p < 3; ++p) { b[p] = be[p]; b[3 + p] = ba[p]; }
    };
    auto contract_keys = [&](auto one_vector) {
#pragma unroll
        for (int round = 0; round < 2 * T; ++round) {
            __syncthreads();  // (what lay there has been read)
            if constexpr (!decltype(one_vector)::value) {
                if (round == 0) {
                    xk.zero_past(row0, n);
                    xk.put(tile);
                }
            }
            hand_round();
            if (round + 1 < 2 * T) prepare_keys(round + 1, one_vector);
#pragma unroll
            for (int g = 0; g < G0; ++g) {
                const tr_bf16x8_t x = rows_transposed((g0 + g) * T + round / 2, round % 2);
                tr_f32x16_t& k = ke[g / S::HB];
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    k = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, handed(g, p), k, 0, 0, 0);
                    dw = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, handed(g, 3 + p), dw, 0, 0, 0);
                }
            }
        }
    };
    if (mixed) {
        auto prepare_queries = [&](int t) {  // 32 rows' dZ_q
            tr_f32x16_t gq;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float sd = s_lab[(t0 + t) * 32 + 8 * (i / 4) + 4 * half + (i % 4)] * (zq[t][i] - zk[t][i]);
                gq[i] = c_sim * sd * fmaf(-zq[t][i], zq[t][i], 1.f);
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                tr_bf16x8_t bq[3];
                split_operand(gq, ks, bq);
#pragma unroll
                for (int p = 0; p < 3; ++p) b[3 * ks + p] = bq[p];
            }
        };
        xk.fetch(K, row0, n);  // (the tile's next content)
        prepare_queries(0);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            __syncthreads();
            hand_round();
            if (t + 1 < T) prepare_queries(t + 1);
            else prepare_keys(0, std::false_type{});
#pragma unroll
            for (int g = 0; g < G0; ++g)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    const tr_bf16x8_t x = rows_transposed((g0 + g) * T + t, ks);
#pragma unroll
                    for (int p = 0; p < 3; ++p) dw = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, handed(g, 3 * ks + p), dw, 0, 0, 0);
                }
        }
        contract_keys(std::false_type{});
    } else {
        prepare_keys(0, std::true_type{});
        contract_keys(std::true_type{});
    }
    // (one query vector: its part of Q^T dZ_q is that vector times the sum over the rows, added behind the sums below)
    ssum += __shfl_xor(ssum, 32, 64);
    if (half == 0) s_dq[rg][w * 32 + m] = mixed ? 0.f : c_sim * ssum * fmaf(-hq0, hq0, 1.f);
    cs += __shfl_xor(cs, 32, 64);
    if (half == 0) s_col[rg][w * 32 + m] = cs;
    lsim = wave_sum64(lsim);
    if (lane == 0) s_loss[tid >> 6] = lsim;
    __syncthreads();
    if (S::RG == 8) {  // two waves have a part each: the second block's meets the first one's
        float* const meet = reinterpret_cast<float*>(s_frag) + ct * 32 * 64 + lane;
        if (rg >= 4) {
#pragma unroll
            for (int i = 0; i < 16; ++i) { meet[i * 64] = ke[0][i]; meet[(16 + i) * 64] = dw[i]; }
        }
        __syncthreads();
        if (rg < 4) {
#pragma unroll
            for (int i = 0; i < 16; ++i) { ke[1][i] = meet[i * 64]; dw[i] += meet[(16 + i) * 64]; }
        }
    }
    if (rg < 4) {
        float g[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < S::RG; ++i) g[i / S::HB] += s_dq[i][w * 32 + m];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; i += 4) {
                const uint2 x = *reinterpret_cast<const uint2*>(&s_q[b][32 * ct + 2 * i + 4 * half]);
                dw[i] = fmaf(bf16_lo(x.x), g[b], dw[i]);
                dw[i + 1] = fmaf(bf16_hi(x.x), g[b], dw[i + 1]);
                dw[i + 2] = fmaf(bf16_lo(x.y), g[b], dw[i + 2]);
                dw[i + 3] = fmaf(bf16_hi(x.y), g[b], dw[i + 3]);
            }
        float* const out = dw_part + (int64_t)blockIdx.x * 3 * HATA_D * R + (32 * ct + 4 * half) * R + col;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int at = (8 * (i / 4) + i % 4) * R;
            out[at] = one_query ? ke[0][i] + ke[1][i] : ke[0][i];
            out[HATA_D * R + at] = dw[i];
            if (!one_query) out[2 * HATA_D * R + at] = ke[1][i];
        }
    }
    // (everybody has written s_col and s_loss: the rounds above have barriers)
    for (int i = tid; i < 2 * COLS; i += THREADS) {
        const int b = i / COLS, jc = i % COLS;
        float t = 0.f;
#pragma unroll
        for (int g = 0; g < S::HB; ++g) t += s_col[b * S::HB + g][jc];
        if (first + b < n_blocks) colsum_part[(int64_t)(first + b) * R + blockIdx.y * COLS + jc] = t;
    }
    if (tid == 0) {  // (the similarity partial of column group y; the groups are summed later)
        float t = 0.f;
        for (int i = 0; i < WAVES; ++i) t += s_loss[i];
        loss_part[blockIdx.y * ((n_blocks + 1) / 2) + blockIdx.x] = t;
        double f = 0.0;
        for (int i = 0; i < WAVES; ++i) f += s_red[i];
        if (wg < GramPiece<R>::PIECES) fro_part[wg] = f;
    }
}

// The same for batches of more than a round of workgroups: grid = (pairs / stages, groups of 32 hash columns), a workgroup goes through
// `stages` pairs of blocks one after the other, a wave through a tile of 32 rows of each, and keeps the sums in registers for a run: up
// to run_len pairs (a share of `stages`, at most TR_KEPT).  The partial of a run lies in its last pair's place.  Only K^T E has a factor per
// query, so where the query changes inside a run it alone is stored, in the place of the last pair of the query that ends, and the rest
// stays in registers (both stored there, and the update one such pair after the other: 960 blocks, r = 128, a query every 23 blocks 80 us, 69 so;
// every 2 blocks 132 and 95, 1920 blocks at r = 32 147 and 82).
//
// Whether a tile holds one query vector is a wave's own matter here; where one does not, the wave takes it and the rest of the run the
// general way, whose sums are the same (the run again from its start, as it was: 256 blocks, r = 128, another vector in the last row of every
// second pair 33.8 us a step, 29.6 so; 960 blocks, every fourth pair 89 and 67, none 64).
//
// What bounds it: a tile is 72 matrix instructions (48 of them the contractions, at the rate these sustain), 500 of the vector ALU
// and 40 KB through LDS, 5 us for the eight waves together.  So the waves have nothing to wait for each other for until a run's sums are
// complete: a wave stages its rows itself, the next tile's under this one's products, makes half of its values under the other half's
// products, and holds the sums for all 128 channels, which meet in LDS at the end (3 us, which is why small batches take the form
// above).  In step with each other, handing the values round through LDS, the waves took 7 us a tile.  us a step, one query vector a
// block / others, the form above with 64 columns / this: r = 128 256 blocks 28.5 / 35.5 -> 27.2 / 34.7, 960 blocks 86 / 108 -> 64 / 83; r = 256
// 256 blocks 52 -> 46, 960 153 / 195 -> 112 / 151; r = 32 960 blocks 42 -> 34.
template <int R>
__global__ __launch_bounds__(TrainShape<32>::THREADS) void train_grad_runs_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const float* __restrict__ s, const float* __restrict__ W,
    int n, int n_blocks, int stages, int run_len, float sigma, float c_sim, const int32_t* __restrict__ block_group, int n_groups,
    float* __restrict__ dw_part, float* __restrict__ colsum_part, float* __restrict__ loss_part, double* __restrict__ gram,
    double* __restrict__ fro_part, float* __restrict__ W_old) {
    using S = TrainShape<32>;
    constexpr int WAVES = S::WAVES;
    // the waves' tiles, K's and Q's in rotation (the next K's, once Q's has been looked at); piece j of row i lies in the place of piece j ^ (i & 15), so that 16 lanes that
    // read a piece of a row each meet in no bank
    __shared__ __attribute__((aligned(16))) uint4 s_tile[WAVES][2][32 * 16];
    __shared__ __attribute__((aligned(16))) uint4 s_weights[8][3][64];  // operand fragments: the planes of the weights, by channel step
    __shared__ __attribute__((aligned(16))) uint16_t s_q[WAVES][HATA_D];  // the tile's query
    __shared__ __attribute__((aligned(16))) float s_lab[WAVES][32];
    __shared__ float s_col[TR_KEPT][WAVES][32];  // per hash column: sums of h(k_n) over a tile
    static_assert(TR_KEPT >= 2, "the first queries' projections in parts, before that");
    __shared__ float s_loss[WAVES];
    __shared__ double s_red[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, rg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 31, half = lane >> 5;
    const int n_pairs = (n_blocks + 1) / 2, p0 = blockIdx.x * stages, p1 = min(p0 + stages, n_pairs);
    const int col = blockIdx.y * 32 + m;
    const int wg = blockIdx.y * gridDim.x + blockIdx.x;
    const bool has_piece = wg < GramPiece<R>::PIECES;
    auto piece_sum = [&]() {
        double f = 0.0;
        for (int i = 0; i < WAVES; ++i) f += s_red[i];
        return f;
    };
    if (p0 >= n_pairs) {  // (small batches have workgroups for the pieces alone)
        if (has_piece) {
            const double f = gram_piece<R>(W, wg, tid, gram, W_old);
            if (lane == 0) s_red[rg] = f;
            __syncthreads();
            if (tid == 0) fro_part[wg] = piece_sum();
        }
        return;
    }
    // (addresses made from it are made where they are used, not in front of the loops and kept in registers)
    auto fresh_lane = [&]() {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    // Rows of X into a tile, past n the last row: eight instructions of four rows, a lane 16 bytes, which land at the
    // instruction's base + 16 lane.  (Instructions rather than the compiler's builtin, which would make every later
    // read of LDS wait for all of them; landed() does.)
    auto request_tile = [&](const uint16_t* X, int row0, uint4* dst) {
        const int l = fresh_lane();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int row = 4 * j + (l >> 4);
            const uint16_t* const g = X + (int64_t)min(row0 + row, n - 1) * HATA_D + ((l & 15) ^ (row & 15)) * 8;
            const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(dst + j * 64));
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(base), "v"(g) : "memory", "m0");
        }
    };
    auto landed = []() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    auto read_done = []() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };  // (what is requested next may take the place of what was read)
    auto row_of = [&](int p) { return p * TR_PAIR + 32 * rg; };
    auto tile_of = [&](int p) { return &s_tile[rg][p & 1][0]; };
    auto zero_past_n = [&](int row0, uint4* t) {  // rows past n count as zeros
        const int l = fresh_lane();
#pragma clang loop unroll(disable)
        for (int j = 0; j < 8; ++j)
            if (row0 + 4 * j + (l >> 4) >= n) t[j * 64 + l] = make_uint4(0, 0, 0, 0);
    };
    request_tile(K, row_of(p0), tile_of(p0));
    request_tile(Q, row_of(p0), tile_of(p0 + 1));
    // the blocks of the next stages with another query than the stage's first block has, a bit each (those past the last block: none)
    auto other_queries = [&](int p) {
        const int own = block_query(block_group, 2 * p, n_groups), b = 2 * p + (lane & (2 * TR_KEPT - 1));
        const int id = block_query(block_group, min(b, n_blocks - 1), n_groups);
        return (uint32_t)__builtin_amdgcn_ballot_w64(b < n_blocks && id != own && lane < 2 * TR_KEPT);
    };
    uint32_t others = other_queries(p0);
    const float nsl = -sigma * TR_LOG2E;
    // The last tile's query, its piece lane % 16 (in s_q too), and its hash values: of the first stage it mostly is the one of the block's first row.
    // A channel step of the planes of the column group's weights by each wave, and of the projections of the two blocks' first rows
    uint4 query = *reinterpret_cast<const uint4*>(Q + (int64_t)min(p0 * TR_PAIR + (rg >> 2) * TR_ROWS, n - 1) * HATA_D + (lane & 15) * 8);
    float hq0;
    {
        const uint4 x = *reinterpret_cast<const uint4*>(Q + (int64_t)min(p0 * TR_PAIR + (m & 1) * TR_ROWS, n - 1) * HATA_D + rg * 16 + 8 * half);
        float wv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) wv[e] = W[(int64_t)(rg * 16 + 8 * half + e) * R + col];
        uint32_t f[3][4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) split3_pair(wv[2 * e2], wv[2 * e2 + 1], f[0][e2], f[1][e2], f[2][e2]);
#pragma unroll
        for (int p = 0; p < 3; ++p) s_weights[rg][p][lane] = make_uint4(f[p][0], f[p][1], f[p][2], f[p][3]);
        tr_f32x16_t z;  // row 0: the first block's, row 1: the second one's
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
#pragma unroll
        for (int p = 0; p < 3; ++p)
            z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(tr_bf16x8_t, x), __builtin_bit_cast(tr_bf16x8_t, make_uint4(f[p][0], f[p][1], f[p][2], f[p][3])), z, 0, 0, 0);
        if (half == 0) {
            s_col[0][rg][m] = z[0];
            s_col[1][rg][m] = z[1];
        }
        __syncthreads();
        float part[WAVES];
#pragma unroll
        for (int i = 0; i < WAVES; ++i) part[i] = s_col[rg >> 2][i][m];
        hq0 = relaxed_sign(((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7])), nsl);
        if (lane < 16) *reinterpret_cast<uint4*>(&s_q[rg][8 * lane]) = query;
    }
    float lsim = 0.f;  // similarity
    auto product = [](tr_bf16x8_t x, tr_bf16x8_t y, tr_f32x16_t& sum) { sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, sum, 0, 0, 0); };
    // Z (32 rows x 32 columns) = X . W: result register ri of lane (m, half) holds row 8 (ri / 4) + 4 half + ri % 4, column m.
    // x(kk): channels 16 kk + 8 half ... of row m
    auto project = [&](auto x) {
        const int l = fresh_lane();
        tr_f32x16_t z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            if (kk == 4) __builtin_amdgcn_sched_barrier(0);  // (sixteen operands at a time, not all of them: registers)
            const tr_bf16x8_t a = x(l, kk);
#pragma unroll
            for (int p = 0; p < 3; ++p) product(a, __builtin_bit_cast(tr_bf16x8_t, s_weights[kk][p][l]), z);
        }
        return z;
    };
    auto project_tile = [&](const uint4* t) {
        return project([&](int l, int kk) { return __builtin_bit_cast(tr_bf16x8_t, t[(l & 31) * 16 + ((2 * kk + (l >> 5)) ^ (l & 15))]); });
    };
    // X transposed: 16 rows (slot (half, j) of the operand <-> row 8 (j / 4) + 4 half + j % 4), 32 channels.  This lane
    // reads channels 32 ct + 16 (m / 16) + 4 (lane % 4) ... of row 16 ks + 4 half + lane % 16 / 4, and of 8 rows on (lds_read_transposed)
    auto rows_transposed = [](const uint4* t, int l, int ks, int ct) {
        const int row = 4 * (l >> 5) + (l & 15) / 4, piece = 2 * (l >> 4 & 1) + (l & 3) / 2;
        const uint16_t* const p = reinterpret_cast<const uint16_t*>(t) + 4 * (l & 1);
        const uint2 lo = lds_read_transposed(p + ((16 * ks + row) * 16 + ((4 * ct + piece) ^ row)) * 8);
        const uint2 hi = lds_read_transposed(p + ((16 * ks + row + 8) * 16 + ((4 * ct + piece) ^ (row + 8))) * 8);
        return __builtin_bit_cast(tr_bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
    };
    auto label_of = [&](int l, int i) { return s_lab[rg][8 * (i / 4) + 4 * (l >> 5) + i % 4]; };
    // What both ways have in common: the tile's K and Q there, its labels, K's projection (then h(k)); requested: Q is too
    auto begin_tile = [&](int p, bool requested, bool with_piece, tr_f32x16_t& zk) {
        const int row0 = row_of(p);
        uint4 *const t = tile_of(p), *const tq = tile_of(p + 1);
        landed();
        const float lab = s[min(row0 + m, n - 1)];
        if (!requested) {
            read_done();
            request_tile(Q, row0, tq);
        }
        if (row0 + 32 > n) zero_past_n(row0, t);
        zk = project_tile(t);
        if (with_piece) {
            const double f = gram_piece<R>(W, wg, 64 * rg + fresh_lane(), gram, W_old);
            if (lane == 0) s_red[rg] = f;
        }
        if (half == 0) s_lab[rg][m] = row0 + m < n ? lab : 0.f;
        landed();
        if (row0 + 32 > n) zero_past_n(row0, tq);
        __builtin_amdgcn_wave_barrier();  // (LDS serves a wave's accesses in order)
    };
    auto squash = [&](tr_f32x16_t& z) {
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = relaxed_sign(z[i], nsl);
    };
    __syncthreads();
    // accumulators: channel 32 ct + 8 (ri / 4) + 4 half + ri % 4, this lane's column
    tr_f32x16_t ke[4], dw[4];  // of a query, K^T E;  of the run, whoever's its rows are, Q^T dZ_q - K^T (A E)
    auto clear = [](tr_f32x16_t (&x)[4]) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) x[ct][i] = 0.f;
    };
#pragma clang loop unroll(disable)
    for (int p = p0, limit = p0; p < p1;) {
        if (p == limit) {
            limit = min(limit + run_len, p1);
            clear(dw);
        }
        clear(ke);
        const bool one_query = (others & 2u) == 0;
        const int pe = one_query ? min(limit, others ? p + (__builtin_ctz(others) >> 1) : limit) : p + 1;  // past the query's pairs in the run
        // h(k) of the tile (zk: its projection) and the contractions with it.  Half of the rows' values are made under the products of the
        // other half: a wave issues a product and then what fits beside it.
        auto contract_keys = [&](const uint4* t, const tr_f32x16_t& zk, auto hash_of_key, auto hash_of_query, float& ssum, float& cs) {
            const int l = fresh_lane();
            uint32_t be[2][3][4], ba[2][3][4];  // the planes of 16 rows' E and -A E
            auto prepare = [&](int ks, int e2) {  // two values
                float e[2], ae[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int i = 8 * ks + 2 * e2 + j;
                    // (half of dL/dh: h' = (1 - h^2) / 2)
                    const float hk = hash_of_key(zk[i]), diff = hash_of_query(i) - hk, sd = label_of(l, i) * diff;
                    cs += hk;  // (rows past n are zero: h = 0)
                    e[j] = fmaf(-hk, hk, 1.f);
                    ae[j] = -c_sim * sd * e[j];
                    lsim = fmaf(sd, diff, lsim);
                    ssum += sd;
                }
                split3_pair(e[0], e[1], be[ks][0][e2], be[ks][1][e2], be[ks][2][e2]);
                split3_pair(ae[0], ae[1], ba[ks][0][e2], ba[ks][1][e2], ba[ks][2][e2]);
            };
            auto plane = [](const uint32_t (&x)[4]) { return __builtin_bit_cast(tr_bf16x8_t, make_uint4(x[0], x[1], x[2], x[3])); };
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) prepare(0, e2);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) {
                    __builtin_amdgcn_sched_barrier(0);
                    const tr_bf16x8_t x = rows_transposed(t, l, ks, ct);
                    if (ks == 0) prepare(1, ct);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        product(x, plane(be[ks][i]), ke[ct]);
                        product(x, plane(ba[ks][i]), dw[ct]);
                    }
                    if (ks == 0) {
#pragma unroll
                        for (int i = 0; i < 6; ++i) {
                            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);  // a product
                            __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);  // vector instructions
                        }
                    }
                }
            }
        };
        int i = p;
        bool general = false;
        {
            float sum_q = 0.f;  // of dZ_q, which the query has yet to be multiplied with
            // one product for 32 channels: the query in the first three places of the contraction, the planes of the sums
            auto add_query = [&]() {
                const int l = fresh_lane();
                uint32_t hi, mid, lo;
                split3_pair(l < 32 ? sum_q : 0.f, 0.f, hi, mid, lo);
                const tr_bf16x8_t y = __builtin_bit_cast(tr_bf16x8_t, make_uint4(hi | mid << 16, lo, 0, 0));
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) {
                    const uint32_t x = s_q[rg][32 * ct + (l & 31)];
                    product(__builtin_bit_cast(tr_bf16x8_t, make_uint4(x | x << 16, x, 0, 0)), y, dw[ct]);
                }
                sum_q = 0.f;
            };
#pragma clang loop unroll(disable)
            for (; i < pe; ++i) {
                tr_f32x16_t zk;
                begin_tile(i, i == p, i == p0 && has_piece, zk);
                const uint4* const tq = tile_of(i + 1);
                const uint4 f = tq[lane & 15];  // the first row's piece lane % 16
                uint32_t stray = 0;
                const int l = fresh_lane();
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int row = 4 * j + (l >> 4);
                    const uint4 x = tq[row * 16 + ((l & 15) ^ (row & 15))];
                    const uint32_t differs = (x.x ^ f.x) | (x.y ^ f.y) | (x.z ^ f.z) | (x.w ^ f.w);
                    const uint32_t counts = x.x | x.y | x.z | x.w | (__float_as_uint(s_lab[rg][row]) << 1);  // (a label of -0 is 0)
                    stray |= counts != 0u ? differs : 0u;
                }
                if (__builtin_amdgcn_ballot_w64(stray != 0u) != 0ull) { general = true; break; }
                if (i + 1 < pe) {
                    read_done();
                    request_tile(K, row_of(i + 1), tile_of(i + 1));
                }
                const uint32_t differs = (f.x ^ query.x) | (f.y ^ query.y) | (f.z ^ query.z) | (f.w ^ query.w);
                if (__builtin_amdgcn_ballot_w64(differs != 0u) != 0ull) {
                    add_query();
                    query = f;
                    if (lane < 16) *reinterpret_cast<uint4*>(&s_q[rg][8 * lane]) = f;
                    __builtin_amdgcn_wave_barrier();
                    hq0 = relaxed_sign(project([&](int l, int kk) { return *reinterpret_cast<const tr_bf16x8_t*>(&s_q[rg][16 * kk + 8 * (l >> 5)]); })[0], nsl);
                }
                float ssum = 0.f, cs = 0.f;  // sums of s (h(q) - h(k)) and of h(k)
                contract_keys(tile_of(i), zk, [&](float z) { return relaxed_sign(z, nsl); }, [&](int) { return hq0; }, ssum, cs);
                sum_q += c_sim * (ssum + __shfl_xor(ssum, 32, 64)) * fmaf(-hq0, hq0, 1.f);
                cs += __shfl_xor(cs, 32, 64);
                if (half == 0) s_col[i - p][rg][m] = cs;
            }
            add_query();
        }
        if (general) {  // from the tile that another vector was met in on, whose rows are there
            bool there = true;
#pragma clang loop unroll(disable)
            for (; i < pe; ++i) {
                tr_f32x16_t zk;
                begin_tile(i, there, false, zk);
                there = false;
                squash(zk);
                const uint4* const tq = tile_of(i + 1);
                tr_f32x16_t zq = project_tile(tq), gq;  // then h(q);  the rows' dZ_q
                squash(zq);
                const int l = fresh_lane();
#pragma unroll
                for (int j = 0; j < 16; ++j) gq[j] = c_sim * label_of(l, j) * (zq[j] - zk[j]) * fmaf(-zq[j], zq[j], 1.f);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    tr_bf16x8_t bq[3];
                    split_operand(gq, ks, bq);
#pragma unroll
                    for (int ct = 0; ct < 4; ++ct) {
                        const tr_bf16x8_t x = rows_transposed(tq, l, ks, ct);
#pragma unroll
                        for (int j = 0; j < 3; ++j) product(x, bq[j], dw[ct]);
                    }
                }
                if (i + 1 < pe) {
                    read_done();
                    request_tile(K, row_of(i + 1), tile_of(i + 1));
                }
                float ssum = 0.f, cs = 0.f;
                contract_keys(tile_of(i), zk, [](float h) { return h; }, [&](int j) { return zq[j]; }, ssum, cs);
                cs += __shfl_xor(cs, 32, 64);
                if (half == 0) s_col[i - p][rg][m] = cs;
            }
        }
        // The waves' sums, the first four the first block's, meet in the tiles' place; a wave adds up 16 channels
        __syncthreads();
        const int l = fresh_lane();
        {  // the column sums, by block
            const int block = 2 * (p + rg) + (l >> 5);
            if (p + rg < pe && block < n_blocks) {
                float sum = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) sum += s_col[rg][4 * (l >> 5) + i][l & 31];
                colsum_part[(int64_t)block * R + col] = sum;
            }
        }
        float4* const meet = reinterpret_cast<float4*>(&s_tile[0][0][0]) + l;
        static_assert(sizeof(s_tile) == WAVES * 64 * 64 * 4, "a wave's sums in its tiles' place");
        float* const out = dw_part + (int64_t)(pe - 1) * 3 * HATA_D * R + 16 * rg * R + blockIdx.y * 32;
        auto store = [&](float* to, int i4, float4 x) {  // channels 8 i4 + 4 half ... of the wave's
            float* const at = to + (uint32_t)((8 * i4 + 4 * (l >> 5)) * R + (l & 31));
            at[0] = x.x; at[R] = x.y; at[2 * R] = x.z; at[3 * R] = x.w;
        };
        auto plus = [](float4 x, float4 y) { return make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w); };
        auto hand_over = [&](const tr_f32x16_t (&x)[4]) {
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
                    meet[(rg * 16 + ct * 4 + i4) * 64] = make_float4(x[ct][4 * i4], x[ct][4 * i4 + 1], x[ct][4 * i4 + 2], x[ct][4 * i4 + 3]);
            __syncthreads();
        };
        auto block_sum = [&](int w0, int i4) {  // over the waves of a block
            const float4* const at = meet + (w0 * 16 + 2 * rg + i4) * 64;
            return plus(plus(at[0], at[16 * 64]), plus(at[32 * 64], at[48 * 64]));
        };
        hand_over(ke);
#pragma unroll
        for (int i4 = 0; i4 < 2; ++i4) {
            const float4 x = block_sum(0, i4), y = block_sum(4, i4);
            if (one_query) {
                store(out, i4, plus(x, y));
            } else {
                store(out, i4, x);
                store(out + 2 * HATA_D * R, i4, y);
            }
        }
        if (pe == limit) {
            __syncthreads();
            hand_over(dw);
#pragma unroll
            for (int i4 = 0; i4 < 2; ++i4) store(out + HATA_D * R, i4, plus(block_sum(0, i4), block_sum(4, i4)));
        }
        p = pe;
        if (p == p1) break;
        __syncthreads();  // (the tiles' places are free again)
        request_tile(K, row_of(p), tile_of(p));
        request_tile(Q, row_of(p), tile_of(p + 1));
        others = other_queries(p);
    }
    lsim = wave_sum64(lsim);
    if (lane == 0) s_loss[rg] = lsim;
    __syncthreads();
    if (tid == 0) {  // (the similarity partial of column group y; the groups are summed later)
        float t = 0.f;
        for (int i = 0; i < WAVES; ++i) t += s_loss[i];
        loss_part[blockIdx.y * ((n_pairs + stages - 1) / stages) + blockIdx.x] = t;
        if (has_piece) fro_part[wg] = piece_sum();
    }
}

// dL/dW = sigma * (sum of the partials) + 2 lam W P / ||P||_F, and the SGD update from it; the last block writes
// the loss terms.  64 elements per workgroup of 512 threads: a wave sums an eighth of the partials of each -- K^T E
// times the column's factor, which the workgroup adds up first from the column sums of all blocks (colsum: already added up per
// query) -- and the eighths meet in LDS in a fixed order.  Large batches are bound by reading the partials once (1 KB times r a run of up to four
// pairs, in the caches: at r = 128 8.4 MB for 256 and 512 blocks, 15.7 for 960; more where queries end inside runs) and the column sums by every workgroup, small ones by the round trips to what a wave reads: hence everything of the first 32 blocks
// is requested at once, queries are looked up by 32 blocks (a lane each), and the loss workgroup's waves have 64 columns of a
// share of the blocks each instead of all columns one after the other (one block 6.5 -> 5.8 us, at r = 256 12.7 -> 8.7;
// 960 blocks of four queries, r = 32 15.6 -> 9.4, r = 128 17.1 -> 13.1).
template <bool RUNS>
__global__ __launch_bounds__(TR_UPDATE_WAVES * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void train_update_kernel(
    float* __restrict__ W, float* __restrict__ v, int log2_r, int n_blocks, int n_loss, float sigma, float lam, float c_sim, float c_bal,
    float lr, float momentum, float weight_decay, const float* __restrict__ dw_part, const float* __restrict__ colsum_part,
    const float* __restrict__ colsum, const int32_t* __restrict__ block_group, int n_groups, const double* __restrict__ gram,
    const double* __restrict__ fro_part, const float* __restrict__ W_old, const float* __restrict__ loss_part,
    float* __restrict__ grad, float* __restrict__ loss, int run_len, int runs) {
    constexpr int WAVES = TR_UPDATE_WAVES;
    __shared__ float part[WAVES][64];
    __shared__ double wp_part[WAVES][64];
    __shared__ float s_slice[WAVES][TR_FEW_QUERIES][64], s_sum[TR_FEW_QUERIES][64];  // column sums: a slice's, a query's
    const int tid = threadIdx.x, el = tid & 63, sl = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = 1 << log2_r, count = HATA_D * r, n_pairs = (n_blocks + 1) / 2;
    constexpr int UN = 16;  // runs of pairs of blocks whose sums are in flight together
    const int n_runs = RUNS ? runs : n_pairs, r0 = sl * n_runs / WAVES, r1 = (sl + 1) * n_runs / WAVES;
    const int b0 = 2 * (RUNS ? run_len : 1) * r0, b1 = min(2 * (RUNS ? run_len : 1) * r1, n_blocks);
    // the queries of blocks b .. below e, a lane each (the lanes behind them: the last one's); the rule: all are one query's
    auto queries_from = [&](int b, int e) { return block_query(block_group, max(min(b + el, e - 1), 0), n_groups); };
    auto uniform = [](int ids) { return __builtin_amdgcn_ballot_w64(ids != __builtin_amdgcn_readfirstlane(ids)) == 0ull; };
    // sums of h(k) per query for column j over blocks [b, e), into s_slice[sl][query][el]; the first 32 blocks and their
    // queries requested ahead
    float cx[2 * UN];
    auto request_columns = [&](int j, int b, int e) {
#pragma unroll
        for (int u = 0; u < 2 * UN; ++u) cx[u] = colsum_part[(int64_t)max(min(b + u, e - 1), 0) * r + j];
    };
    auto add_columns = [&](int j, int b, int e, int ids) {
        for (int q = 0; q < n_groups; ++q) s_slice[sl][q][el] = 0.f;
        for (; b < e; b += 2 * UN) {
            if (uniform(ids)) {
                float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < 2 * UN; ++u) x[u & 3] += b + u < e ? cx[u] : 0.f;
                s_slice[sl][__builtin_amdgcn_readfirstlane(ids)][el] += (x[0] + x[1]) + (x[2] + x[3]);
            } else {
                int query = __builtin_amdgcn_readfirstlane(ids);
                float sum = 0.f;
#pragma unroll
                for (int u = 0; u < 2 * UN; ++u) {
                    if (b + u < e) {
                        const int of = __builtin_amdgcn_readlane(ids, u);
                        if (of != query) {
                            s_slice[sl][query][el] += sum;
                            sum = 0.f;
                            query = of;
                        }
                        sum += cx[u];
                    }
                }
                s_slice[sl][query][el] += sum;
            }
            if (b + 2 * UN < e) {
                request_columns(j, b + 2 * UN, e);
                ids = queries_from(b + 2 * UN, min(b + 4 * UN, e));
            }
        }
    };
    // (everything a wave reads first is requested before any of it is waited for)
    double f2 = 0.0, fp[2 * HATA_D / 64];
    if (sl == 0) {
#pragma unroll
        for (int i = 0; i < 2 * HATA_D / 64; ++i) fp[i] = fro_part[el + 64 * i];
    }
    auto fro_norm = [&]() {  // (wave 0)
#pragma unroll
        for (int i = 0; i < 2 * HATA_D / 64; ++i) f2 += fp[i];
        return (float)sqrt(fmax(wave_sum64_f64(f2) + (double)r, 0.0));
    };
    if ((int)blockIdx.x * 64 < count) {  // (count is a multiple of 64; the last block is past it)
        const int e0 = blockIdx.x * 64, e = e0 + el, j = e & (r - 1);
        const float* const dp = dw_part + e;
        int ids = queries_from(b0, min(b0 + 2 * UN, b1));
        if (!colsum) request_columns(j, b0, b1);
        float ke[UN], dw[UN];
        // what the last pairs of runs i, i + 1, ... hold: the run's sums, of K^T E those of its last query
        auto fetch = [&](int i) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int run = max(min(i + u, r1 - 1), 0);
                const float* at = dp + (int64_t)(RUNS ? min((run + 1) * run_len, n_pairs) - 1 : run) * 3 * count;
                ke[u] = at[0];
                dw[u] = at[count];
            }
        };
        // The pairs of runs i .. i + UN - 1, a lane each: the queries of its blocks, whether it is its run's last, whether its query ends with it
        static_assert(UN * TR_KEPT <= 64, "a lane a pair");
        struct RunPairs { int q0, q1; bool live, last, ends; int run_query; };
        auto pairs_from = [&](int i) {
            int l = el;
            asm volatile("" : "+v"(l));  // (made here, not in front of the loops)
            const int own = i * run_len + l, p_end = min(min(i + UN, r1) * run_len, n_pairs);
            auto query_of = [&](int k) { return block_query(block_group, max(min(min(2 * own + k, 2 * p_end - 1), n_blocks - 1), 0), n_groups); };
            const int q0 = query_of(0), q1 = query_of(1), q2 = query_of(2), q3 = query_of(3);
            const int run_end = min((i + (l & (UN - 1)) + 1) * run_len, p_end);  // of run i + lane % UN, whose last pair's first query is
            const int run_query = block_query(block_group, max(2 * run_end - 2, 0), n_groups);
            return RunPairs{q0, q1, own < p_end, (l + 1) % run_len == 0 || own + 1 >= p_end, q1 != q0 || q2 != q0 || q3 != q0, run_query};
        };
        RunPairs next_pairs;
        if constexpr (RUNS) next_pairs = pairs_from(r0);
        fetch(r0);
        constexpr int NG = HATA_D / WAVES;
        float wo[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) wo[i] = W_old[(sl * NG + i) * r + j];
        const float w0 = W[e], v0 = v[e];
        // (the workgroup's elements are one channel's, or at r = 32 two channels')
        const double* const g_lo = gram + (e0 >> log2_r) * HATA_D + sl * NG;
        const double* const g_hi = gram + ((e0 + 63) >> log2_r) * HATA_D + sl * NG;
        const bool hi = (e >> log2_r) != (e0 >> log2_r);
        if (!colsum) {
            add_columns(j, b0, b1, ids);
            __syncthreads();
            for (int q = sl; q < n_groups; q += WAVES) {
                float t = 0.f;
#pragma unroll
                for (int i = 0; i < WAVES; ++i) t += s_slice[i][q][el];
                s_sum[q][el] = t;
            }
            __syncthreads();
        }
        auto factor_of = [&](int q) { return c_bal * (colsum ? colsum[(int64_t)q * r + j] : s_sum[q][el]); };
        float gp[4] = {0.f, 0.f, 0.f, 0.f};
        for (int p = r0; p < (RUNS ? r0 : r1); p += UN) {  // (a run: a pair of blocks)
            if (p != r0) {
                ids = queries_from(2 * p, min(2 * (p + UN), b1));
                fetch(p);
            }
            if (uniform(ids)) {
                const float fc = factor_of(__builtin_amdgcn_readfirstlane(ids));
#pragma unroll
                for (int u = 0; u < UN; ++u) gp[u & 3] += p + u < r1 ? fmaf(fc, ke[u], dw[u]) : 0.f;
            } else {
                float f0[UN], f1[UN], k1[UN];
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    const int q0 = __builtin_amdgcn_readlane(ids, 2 * u), q1 = __builtin_amdgcn_readlane(ids, 2 * u + 1);
                    f0[u] = factor_of(q0);
                    f1[u] = k1[u] = 0.f;
                    if (q1 != q0) {
                        f1[u] = factor_of(q1);
                        k1[u] = dp[((int64_t)(p + u) * 3 + 2) * count];
                    }
                }
#pragma unroll
                for (int u = 0; u < UN; ++u) gp[u & 3] += p + u < r1 ? fmaf(f1[u], k1[u], fmaf(f0[u], ke[u], dw[u])) : 0.f;
            }
        }
        for (int i = r0; i < (RUNS ? r1 : r0); i += UN) {
            const RunPairs own = next_pairs;
            const int first = __builtin_amdgcn_readfirstlane(own.q0);
            if (__builtin_amdgcn_ballot_w64(own.q0 != first || own.q1 != first) == 0ull) {
                const float fc = factor_of(first);
#pragma unroll
                for (int u = 0; u < UN; ++u) gp[u & 3] += i + u < r1 ? fmaf(fc, ke[u], dw[u]) : 0.f;
                if (i + UN < r1) {
                    next_pairs = pairs_from(i + UN);
                    fetch(i + UN);
                }
                continue;
            }
            {
                float f[UN];  // of the query that a run ends with (of two the first one)
#pragma unroll
                for (int u = 0; u < UN; ++u) f[u] = factor_of(__builtin_amdgcn_readlane(own.run_query, u));
#pragma unroll
                for (int u = 0; u < UN; ++u) gp[u & 3] += i + u < r1 ? fmaf(f[u], ke[u], dw[u]) : 0.f;
            }
            // What else runs with several queries hold: a place where a query ends inside the run, and of pairs of two queries the second one's.
            // UB of them in flight together, behind no branch (past the last one that one again)
            constexpr int UB = 8;
            float k[UB], f[UB];
            auto request = [&](unsigned long long& left, int queries, int part_of_place, int u0, int u1) {
#pragma unroll
                for (int u = u0; u < u1; ++u) {
                    const int p = left ? __builtin_ctzll(left) : 0;
                    if (left & (left - 1)) left &= left - 1;
                    k[u] = dp[((int64_t)(i * run_len + p) * 3 + part_of_place) * count];
                    f[u] = factor_of(__builtin_amdgcn_readlane(queries, p));
                }
            };
            auto add = [&](int u0, int u1, int n) {
#pragma unroll
                for (int u = u0; u < u1; ++u) gp[u & 3] += u - u0 < n ? f[u] * k[u] : 0.f;
            };
            unsigned long long places = __builtin_amdgcn_ballot_w64(own.live && own.ends && !own.last),
                               mixed = __builtin_amdgcn_ballot_w64(own.live && own.q1 != own.q0);
            int n_places = __builtin_popcountll(places), n_mixed = __builtin_popcountll(mixed);
            if (i + UN < r1) next_pairs = pairs_from(i + UN);
            if (n_places <= 2 && n_mixed <= 2) {
                if (n_places + n_mixed > 0) {
                    request(places, own.q0, 0, 0, 2);
                    request(mixed, own.q1, 2, 2, 4);
                    add(0, 2, n_places);
                    add(2, 4, n_mixed);
                }
            } else {
#pragma clang loop unroll(disable)
                for (; n_places > 0; n_places -= UB) {
                    request(places, own.q0, 0, 0, UB);
                    add(0, UB, n_places);
                }
#pragma clang loop unroll(disable)
                for (; n_mixed > 0; n_mixed -= UB) {
                    request(mixed, own.q1, 2, 0, UB);
                    add(0, UB, n_mixed);
                }
            }
            if (i + UN < r1) fetch(i + UN);
        }
        double wp = 0.0;
#pragma unroll
        for (int i = 0; i < NG; ++i) wp = fma(hi ? g_hi[i] : g_lo[i], (double)wo[i], wp);
        part[sl][el] = (gp[0] + gp[1]) + (gp[2] + gp[3]);
        wp_part[sl][el] = wp;
        __syncthreads();
        if (sl == 0) {
            const float fro = fro_norm();
            float g = 0.f;
#pragma unroll
            for (int i = 0; i < WAVES; ++i) g += part[i][el];
            wp = -(double)w0;
#pragma unroll
            for (int i = 0; i < WAVES; ++i) wp += wp_part[i][el];
            g *= sigma;
            if (fro > 0.f) g += lam * 2.f * (float)wp / fro;
            if (grad) grad[e] = g;
            const float vn = fmaf(momentum, v0, fmaf(weight_decay, w0, g));
            v[e] = vn;
            W[e] = fmaf(-lr, vn, w0);
        }
        return;
    }
    // similarity: sum of the workgroup partials; balance: squared norm of the column sums
    float ls = 0.f, lb = 0.f;
    for (int i = tid; i < n_loss; i += WAVES * 64) ls += loss_part[i];
    if (colsum) {
        for (int j = tid; j < r * n_groups; j += 16 * WAVES * 64) {
            float x[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) x[u] = colsum[min(j + u * WAVES * 64, r * n_groups - 1)];
#pragma unroll
            for (int u = 0; u < 16; ++u) lb = j + u * WAVES * 64 < r * n_groups ? fmaf(x[u], x[u], lb) : lb;
        }
    } else {
        // a wave: 64 columns of a share of the blocks
        const int cols = (r + 63) / 64, share = WAVES / cols, grp = sl % cols, at = sl / cols;
        const int first = at * n_blocks / share, last = (at + 1) * n_blocks / share, j = min(grp * 64 + el, r - 1);
        const int ids = queries_from(first, min(first + 2 * UN, last));
        request_columns(j, first, last);
        add_columns(j, first, last, ids);
        __syncthreads();
        for (int i = sl; i < n_groups * cols; i += WAVES) {
            const int q = i / cols, g = i % cols;
            float t = 0.f;
            for (int k = 0; k < share; ++k) t += s_slice[k * cols + g][q][el];
            if (g * 64 + el < r) lb = fmaf(t, t, lb);
        }
    }
    ls = wave_sum64(ls);
    lb = wave_sum64(lb);
    if (el == 0) { part[0][sl] = ls; part[1][sl] = lb; }
    const float fro = sl == 0 ? fro_norm() : 0.f;
    __syncthreads();
    if (tid == 0) {
        ls = lb = 0.f;
        for (int i = 0; i < WAVES; ++i) { ls += part[0][i]; lb += part[1][i]; }
        loss[0] = c_sim * ls;
        loss[1] = c_bal * lb;
        loss[2] = lam * fro;
    }
}

// ---- label builder (App. B.1, steps 3-4) ----------------------------------------------------------
// Rank of a pair = number of pairs with a larger score, or an equal score and a lower index; the first n_pos
// ranks (a tenth of the pairs) get 20 .. 1 in equal steps, the others -1.  Counting every pair against every
// other one costs m^2 compares (571 us at m = 8192), and nine pairs in ten only need to know that they
// are not among the first tenth.  So three launches: the scores, with a coarse histogram of them; from the
// histogram the bin the n_pos-th score lies in -- everything below it is -1, everything from it up goes into a
// candidate list, in any order; ranks by counting inside that list (a hundredth of the compares where the scores
// spread over the bins; m^2 again if they all fall into one).  14 us at m = 8192.
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

// ranks inside the candidate list: LB_RANKED * PER candidates per workgroup and turn, a lane for PER of them in every sixteen, each counted
// by 64 groups of lanes over a 64th of the list; the histogram is cleared for the next call.  Bound by the compares' instructions where
// workgroups are few: 64 candidates a workgroup, each wave handing a sixteenth of the list round as scalars, were 27 workgroups at 8192 keys
// and 9.2 us, these 104 take 5.1.  Long lists are bound by their reads, the whole of it a workgroup: PER = 4 from LB_LONG expected on (us a
// call, scalars / one / four a lane: 52000 keys 49.4 / 36.4 / 35.2, 100000 87 / 81 / 59, 1000000 4450 / 4760 / 2380; all 65536 scores equal 2010 / 2400 / 1060).
#define LB_RANKED 16
#define LB_LONG 5120
template <int PER>
__global__ __launch_bounds__(1024) void train_labels_kernel(const LabelCand* __restrict__ cand, const uint32_t* __restrict__ n_cand,
                                                            int n_pos, uint32_t* __restrict__ bins, float* __restrict__ s) {
    __shared__ int s_rank[16][LB_RANKED * PER];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, own = lane % LB_RANKED;
    if (blockIdx.x == gridDim.x - 1)
        for (int i = tid; i < LB_COPIES * LB_BINS; i += 1024) bins[i] = 0;
    const int nc = (int)*n_cand;
    for (int c0 = blockIdx.x * LB_RANKED * PER; c0 < nc; c0 += gridDim.x * LB_RANKED * PER) {
        unsigned long long key[PER];
        uint32_t row[PER];
        int rank[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const LabelCand me = cand[min(c0 + own + LB_RANKED * k, nc - 1)];
            key[k] = me.key; row[k] = me.row; rank[k] = 0;
        }
        constexpr int UN = 8;  // entries of a lane in flight together
        for (int j0 = tid / LB_RANKED; j0 < nc; j0 += 64 * UN) {
            LabelCand o[UN];
#pragma unroll
            for (int t = 0; t < UN; ++t) o[t] = cand[min(j0 + 64 * t, nc - 1)];
#pragma unroll
            for (int t = 0; t < UN; ++t)
#pragma unroll
                for (int k = 0; k < PER; ++k)
                    if constexpr (PER > 1)  // (no branches: with them 41.6 us at 52000 keys)
                        rank[k] += (int)(j0 + 64 * t < nc) & ((int)(o[t].key > key[k]) | ((int)(o[t].key == key[k]) & (int)(o[t].row < row[k])));
                    else
                        rank[k] += j0 + 64 * t < nc && (o[t].key > key[k] || (o[t].key == key[k] && o[t].row < row[k])) ? 1 : 0;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            rank[k] += __shfl_xor(rank[k], 16, 64);
            rank[k] += __shfl_xor(rank[k], 32, 64);
            if (lane < LB_RANKED) s_rank[wave][LB_RANKED * k + lane] = rank[k];
        }
        __syncthreads();
        if (tid < LB_RANKED * PER && c0 + tid < nc) {
            uint32_t at = row[0];
            int sum = 0;
#pragma unroll
            for (int k = 1; k < PER; ++k) at = tid / LB_RANKED == k ? row[k] : at;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += s_rank[i][tid];
            s[at] = sum < n_pos ? rank_label(sum, n_pos) : -1.f;
        }
        __syncthreads();
    }
}

}  // namespace hata

namespace {
constexpr size_t kAlignT = 256;
inline size_t align_up_t(size_t x) { return (x + kAlignT - 1) / kAlignT * kAlignT; }
struct TrainPlan { int n_wgs_max; size_t off_colsum, off_cs, off_dw, off_loss, off_gram, off_fro, off_old, off_scores, off_bins, off_ncand, off_cand, total; };
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
    const size_t pairs = ((size_t)p->n_wgs_max + 1) / 2;
    p->off_dw = o;     o = align_up_t(o + pairs * 3 * f->d * f->r * 4);
    p->off_loss = o;   o = align_up_t(o + (pairs * 4 > TR_ONE_ROUND ? pairs * 4 : TR_ONE_ROUND) * 4);
    p->off_gram = o;   o = align_up_t(o + (size_t)f->d * f->d * 8);
    p->off_fro = o;    o = align_up_t(o + (size_t)f->d * 2 * 8);
    p->off_old = o;    o = align_up_t(o + (size_t)f->d * f->r * 4);
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
    c->gram = (double*)(w + p.off_gram);
    c->fro_part = (double*)(w + p.off_fro);
    c->W_old = (float*)(w + p.off_old);
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
    const bool few = n_wgs <= TR_FEW_WGS && n_queries <= TR_FEW_QUERIES;
    const float* colsum = few ? nullptr : ctx->colsum;
    // The gradient launch.  A workgroup per pair of blocks and 32 hash columns where that is at most one round of the chip, which is through
    // sooner than one of 64 (us a step, one query vector a block / others: one block r = 64 20.3 / 26.4 -> 16.6 / 19.5, r = 256 24.3 / 30.1 ->
    // 20.2 / 23.0; 64 blocks r = 128 23.5 / 29.1 -> 19.9 / 22.6).  Beyond, a workgroup goes through as many pairs as one round takes, in
    // runs of at most TR_KEPT, unless queries that end inside its pairs cost it more than that saves, of which the host knows the number alone
    // (a pair and 64 columns, at r = 32 32 / runs):
    // - queries of less than eight blocks on average: every 3 blocks, r = 64, 1030 blocks 74.0 / 80.0, r = 256, 256 blocks 52.0 / 56.4; the latter
    //   every 7 blocks 47.1 / 50.0, every 9 57.7 / 59.3, which is the worst of them (r = 128, 384 to 1536 blocks, every 7 to 23: 6 to 24 % less)
    // - where two pairs would do, several queries: such an end costs as much there as runs save, so up to four of them, where the second round is
    //   as good as full, and none below.  r = 128, 256 blocks: equal shares 27.8 .. 29.8 / 26.4 .. 27.9, uneven ones 28.4 .. 30.9 / 28.6 .. 30.2 by
    //   where the buffers lie; 192 blocks, uneven 27.5 .. 28.0 / 28.5 .. 29.4; r = 64 512 blocks 29.5 .. 31.1 / 30.1 .. 31.7, 450 30.0 / 31.1; r = 256
    //   128 blocks 35.0 / 34.9, 120 35.2 / 35.6.  One query: r = 128 132 blocks 26.3 / 26.2, 192 27.8 / 27.2; r = 256 128 33.5 / 32.2
    // At least a piece of W W^T each: workgroups behind the pairs have nothing else.
    const int pairs = (n_wgs + 1) / 2, pairs_32 = pairs * (r / 32);
    const bool two_pairs = r > 32 && pairs_32 <= 2 * TR_ONE_ROUND;
    const bool one_stage = pairs_32 <= TR_ONE_ROUND || n_wgs < 8 * n_queries ||
                           (two_pairs && n_queries > (pairs_32 > 2 * TR_ONE_ROUND / 64 * 63 ? 4 : 1));
    const int cols = one_stage && r > 32 && pairs_32 > TR_ONE_ROUND ? 64 : 32, col_groups = r / cols;
    const int least = one_stage ? 1 : (pairs * col_groups + TR_ONE_ROUND - 1) / TR_ONE_ROUND;
    const int runs_each = (least + TR_KEPT - 1) / TR_KEPT, run_len = (least + runs_each - 1) / runs_each, stages = runs_each * run_len;
    const int n_runs = (pairs + run_len - 1) / run_len, n_grad_wgs = (pairs + stages - 1) / stages;
    const int n_grad = n_grad_wgs * col_groups < 2 * HATA_D ? 2 * HATA_D / col_groups : n_grad_wgs;
#define HATA_TRAIN_ONE(RR, CC)                                                                                           \
    hipLaunchKernelGGL((hata::train_grad_kernel<RR, CC>), dim3(n_grad, RR / CC), dim3(hata::TrainShape<CC>::THREADS), 0, \
                       st, q, k, s, W, n, n_wgs, hp->sigma, c_sim, block_query, n_queries, ctx->dw_part,                 \
                       ctx->colsum_part, ctx->loss_part, ctx->gram, ctx->fro_part, ctx->W_old)
#define HATA_TRAIN_CASE(RR)                                                                                                         \
    case RR:                                                                                                                        \
        if (!one_stage)                                                                                                             \
            hipLaunchKernelGGL(hata::train_grad_runs_kernel<RR>, dim3(n_grad, RR / 32), dim3(hata::TrainShape<32>::THREADS), 0, st, \
                               q, k, s, W, n, n_wgs, stages, run_len, hp->sigma, c_sim, block_query, n_queries, ctx->dw_part,       \
                               ctx->colsum_part, ctx->loss_part, ctx->gram, ctx->fro_part, ctx->W_old);                             \
        else if (cols == 32)                                                                                                        \
            HATA_TRAIN_ONE(RR, 32);                                                                                                 \
        else                                                                                                                        \
            HATA_TRAIN_ONE(RR, (RR < 64 ? 32 : 64));                                                                                \
        break
    switch (r) {
        HATA_TRAIN_CASE(32);
        HATA_TRAIN_CASE(64);
        HATA_TRAIN_CASE(128);
        HATA_TRAIN_CASE(256);
    }
#undef HATA_TRAIN_CASE
#undef HATA_TRAIN_ONE
    if (!few)
        hipLaunchKernelGGL(hata::train_colreduce_kernel, dim3((r + 63) / 64, n_queries), dim3(TR_REDUCE_WAVES * 64), 0, st,
                           ctx->colsum_part, r, n_wgs, block_query, n_queries, ctx->colsum);
    hipLaunchKernelGGL(run_len > 1 ? hata::train_update_kernel<true> : hata::train_update_kernel<false>, dim3(HATA_D * r / 64 + (loss ? 1 : 0)),
                       dim3(TR_UPDATE_WAVES * 64), 0, st, W, v, __builtin_ctz(r), n_wgs, n_grad_wgs * col_groups,
                       hp->sigma, hp->lam, c_sim, c_bal, hp->lr, hp->momentum, hp->weight_decay, ctx->dw_part,
                       ctx->colsum_part, colsum, block_query, n_queries, ctx->gram, ctx->fro_part, ctx->W_old,
                       ctx->loss_part, grad, loss, run_len, n_runs);
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
    // enough workgroups for twice the expected list, and for short ones of equal scores (they take more turns if it is longer)
    hipLaunchKernelGGL(n_pos > LB_LONG ? hata::train_labels_kernel<4> : hata::train_labels_kernel<1>, dim3(n_pos / (LB_RANKED / 2) + 8), dim3(1024), 0, st,
                       ctx->cand, ctx->n_cand, n_pos, ctx->bins, s);
    const bool ok = hipGetLastError() == hipSuccess;
    ctx->bins_clear = ok && cleared;  // (after a call that failed half-way the next one clears again)
    return ok ? HATA_OK : HATA_EHIP;
}

}  // extern "C"
