// HashEncode kernels (Alg. 2 of the paper): codes = BitPack(Sign(x . W_H)).
//
//   encode_few_kernel      the query heads of a unit and up to eight keys of it; fp64 accumulation (hata_hash.h).
//   encode_bulk_kernel     64 keys per workgroup, fp32 accumulation (prefill, the key-code fill of Alg. 1).
#include "hata_device.h"
#include "hata_hash.h"
#include "hata_internal.h"

namespace hata {

// Bit j of a code goes to word j/32, bit position j%32; bit = (projection >= 0).
// grid = (slices of COLS hash columns, B * Hkv): the workgroup encodes, on its columns, the G query heads of its unit (q
// not null) and n_new[b] <= max_new keys from row start[b] on (K not null; from_seq_len: the one key at row
// start[b] - 1), four vectors at a time, the next four's channels fetched ahead.  Bound by latency, the
// launch and two round trips to memory; a workgroup of 1024 threads per unit (queries) or per key on the vector
// ALU took 4.0 and 11.5 us at 64 units, r = 128, this took 3.9 for both.
// ONE: a launch that has at most one vector a unit, over the vector ALU (hash_one): 64 units, r = 128, a query and a key 0.4 us less
// each, the five stage calls of two layers 51.9 -> 50.1 us.  (Chosen inside the kernel, for a last one behind the fours too, it cost the
// launches of six vectors 0.2 us: their code is fetched anew every time.)
template <int COLS, bool ONE>
__global__ __launch_bounds__(256) void encode_few_kernel(
    const uint16_t* __restrict__ q, uint32_t* __restrict__ qcodes, const uint16_t* __restrict__ K,
    const int32_t* __restrict__ start, const int32_t* __restrict__ n_new, int max_new, int from_seq_len,
    uint32_t* __restrict__ codes, const float* __restrict__ W_H, int Hq, int Hkv, int G, int r, int L_cap,
    int64_t sb, int64_t sh, int64_t sn) {
    constexpr int WPS = COLS / 32;  // code words of a slice
    __shared__ uint32_t s_codes[(16 + 8) * WPS];
    const int tid = threadIdx.x;
    const int u = blockIdx.y, b = u / Hkv, h = u % Hkv;
    HashWeights<COLS> hw;
    hw.fetch(W_H + (int64_t)h * HATA_D * r + blockIdx.x * COLS, r);
    const int nq = q ? G : 0;
    int row0 = 0, nk = 0;  // keys: rows row0 .. row0 + nk - 1 that lie in the cache
    if (K) {
        row0 = from_seq_len ? start[b] - 1 : start[b];
        nk = from_seq_len ? 1 : clampi(n_new[b], 0, max_new);
        if (row0 < 0) { nk = max(nk + row0, 0); row0 = 0; }
        nk = min(nk, L_cap - row0);
    }
    const int nv = nq + max(nk, 0);
    const uint16_t* qu = q + ((int64_t)b * Hq + (int64_t)h * G) * HATA_D;
    const uint16_t* Ku = K + b * sb + h * sh + row0 * sn;
    auto load = [&](int v0, uint4 (&x)[4]) {
        const int v = min(v0 + (tid & 3), nv - 1);
        hash_load_x(v < nq ? qu + v * HATA_D : Ku + (v - nq) * sn, x);
    };
    if (nv <= 0) return;
    uint4 x[4], xn[4];
    load(0, x);
    for (int v0 = 0; v0 < (ONE ? 1 : nv); v0 += 4) {
        if (!ONE && v0 + 4 < nv) load(v0 + 4, xn);
        if constexpr (ONE) hash_one<COLS>(hw, x, s_codes, WPS, v0);
        else hash_pass<COLS>(hw, x, s_codes, WPS, v0, nv);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = xn[i];
    }
    __syncthreads();
    const int Wd = r / 32;
    for (int i = tid; i < nv * WPS; i += 256) {
        const int v = i / WPS, w = blockIdx.x * WPS + i % WPS;
        if (v < nq) qcodes[((int64_t)b * Hq + (int64_t)h * G + v) * Wd + w] = s_codes[i];
        else codes[((int64_t)u * L_cap + row0 + v - nq) * Wd + w] = s_codes[i];
    }
}

// 64 keys per workgroup; thread = (key, word group).  The word group is uniform over a
// wave, so the W_H reads are wave-uniform.  grid = (tiles, Hkv, B).
__global__ __launch_bounds__(256) void encode_bulk_kernel(
    const uint16_t* __restrict__ K, const float* __restrict__ W_H,
    const int32_t* __restrict__ start, const int32_t* __restrict__ n_new,
    uint32_t* __restrict__ codes, int Hkv, int r, int Wd, int L_cap,
    int64_t sb, int64_t sh, int64_t sn) {
    __shared__ float xs[64][HATA_D + 1];
    const int tid = threadIdx.x;
    const int h = blockIdx.y, b = blockIdx.z;
    const int first = start[b];
    const int cnt = n_new[b];
    const int t0 = blockIdx.x * 64;
    if (t0 >= cnt) return;
    const int64_t u = (int64_t)b * Hkv + h;
    // stage the tile: 16 lanes per row, 16 B (8 bf16) per lane
    for (int it = 0; it < 4; ++it) {
        const int row = it * 16 + (tid >> 4);
        const int n = first + t0 + row;
        const int sub = tid & 15;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (t0 + row < cnt && n >= 0 && n < L_cap)
            v = *reinterpret_cast<const uint4*>(K + b * sb + h * sh + (int64_t)n * sn + sub * 8);
        float* dstp = &xs[row][sub * 8];
        dstp[0] = bf16_lo(v.x); dstp[1] = bf16_hi(v.x);
        dstp[2] = bf16_lo(v.y); dstp[3] = bf16_hi(v.y);
        dstp[4] = bf16_lo(v.z); dstp[5] = bf16_hi(v.z);
        dstp[6] = bf16_lo(v.w); dstp[7] = bf16_hi(v.w);
    }
    __syncthreads();
    const int key = tid & 63;
    const int n = first + t0 + key;
    const bool live = (t0 + key < cnt) && n >= 0 && n < L_cap;
    const int wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int w = wg; w < Wd; w += 4) {
        float acc[32];
#pragma unroll
        for (int c = 0; c < 32; ++c) acc[c] = 0.f;
        const float* wp = W_H + (int64_t)h * HATA_D * r + w * 32;
        for (int i = 0; i < HATA_D; ++i) {
            const float xv = xs[key][i];
#pragma unroll
            for (int c = 0; c < 32; ++c) acc[c] = fmaf(xv, wp[(int64_t)i * r + c], acc[c]);
        }
        uint32_t word = 0;
#pragma unroll
        for (int c = 0; c < 32; ++c) word |= (acc[c] >= 0.f ? 1u : 0u) << c;
        if (live) codes[(u * L_cap + n) * Wd + w] = word;
    }
}

// ---------------------------------------------------------------------------------------
// Prefill key-code writer on the matrix cores (Alg. 1: K_H = HashEncode(K) during the prefill).
//
// The projection [keys, 128] x [128, r] is a dense contraction, so it runs on MFMA
// (v_mfma_f32_32x32x16_bf16).  K is bf16 already; the fp32 weights are split exactly into
// three bf16 planes (hi + mid + lo carries all 24 mantissa bits), every bf16 x bf16 product is
// exact in fp32, and only the fp32 accumulation rounds (~1e-6 relative) -- which is what keeps
// the sign bits equal to an exact evaluation outside a |projection| < ~1e-5 band.
//
// Mapping: M = 32 hash columns (wave w owns columns [32 w, 32 w + 32), i.e. code word w),
// N = 32 keys, K = channels.  A wave keeps its weight fragments (3 planes x 8 channel steps) in
// registers for the whole launch; key rows are staged through LDS 128 at a time (64 in the fill and at r = 32) with coalesced
// 128-bit loads (next stage prefetched into registers) and read back in the operand layout
// (lane = key, 16 B of consecutive channels).  In the 32x32 result a lane holds 16 hash columns of
// ONE key, so the sign bits are packed inside the lane and joined with the other half-wave.
// grid = (key blocks, Hkv, B); R / 32 waves per workgroup (r = 32, 64, 128 or 256).
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
#define HATA_MFMA_PITCH 136   // LDS row pitch in bf16 elements (272 B: rows shift by 4 banks)


// Bit 8 (i / 4) + i % 4: acc[i] >= 0, the complement of the sign bit (a sum of exact products that starts from +0 is
// never -0; the NaN that the matrix cores make of a NaN or of infinities that cancel has its sign bit set, whatever the
// input's was, so such a bit is 0 as in a comparison).  One instruction a value and four to part the groups of four; with two a value, shift and
// insertion, 131072 keys of eight heads took encode_dma_kernel 135.4 us instead of 132.1 (r = 256), 70.8 instead of 68.1 (128).
__device__ __forceinline__ uint32_t sign_bits(const f32x16_t& acc) {
    uint32_t neg = 0;
#pragma unroll
    for (int i = 15; i >= 0; --i) neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[i]), 31);  // 2 neg + sign
    neg = (neg | neg << 8) & 0x00ff00ffu;
    return ~(neg | neg << 4) & 0x0f0f0f0fu;
}

// fp32 weight pair -> the three bf16 planes (hi, mid, lo) whose sum is the weight exactly; two weights per dword
__device__ __forceinline__ void split_weight_pair(float w0, float w1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    uint32_t ph[2], pm[2], pl[2];
    const float wv2[2] = {w0, w1};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float wv = wv2[q];
        ph[q] = f32_to_bf16(wv);
        const float r1 = wv - __uint_as_float(ph[q] << 16);
        pm[q] = f32_to_bf16(r1);
        const float r2 = r1 - __uint_as_float(pm[q] << 16);
        pl[q] = f32_to_bf16(r2);
    }
    hi = ph[0] | (ph[1] << 16);
    mid = pm[0] | (pm[1] << 16);
    lo = pl[0] | (pl[1] << 16);
}

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;

// eight bf16 values (one 16-byte operand fragment) -> fp16
__device__ __forceinline__ f16x8_t bf16x8_to_f16(const uint4 v) {
    const uint32_t x[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        o[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(bf16_lo(x[i]), bf16_hi(x[i])));
    return __builtin_bit_cast(f16x8_t, make_uint4(o[0], o[1], o[2], o[3]));
}

// 16 bytes that nobody reads again
__device__ __forceinline__ uint4 load_once(const uint16_t* p) {
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p)));
}

// FILL: the fused cache fill.  It is bound by the bytes it moves (512 read and 512 written a key), so all of a
// stage's K and V pieces and the rows they go to are requested together, the stores follow when the rows are
// put into LDS, stages are half as long (registers: three waves per SIMD instead of two) and the source is
// read with non-temporal loads, which leave the caches to the rows just written.  Prompts of 8011, 3932, 6057
// and 2712 tokens into a paged cache, eight heads, r = 128: 54.1 us with a load, a store and a table lookup at a
// time, 40.3 with them batched, 35.2 with the loads non-temporal (4.9 TB/s; stores of that kind too: 38.4).
//
// PRESPLIT: the weights come from the planes hata_prepare_weights made, and they are the two scaled
// fp16 planes described at encode_dma_kernel below (two MFMAs per fragment instead of three; the key
// rows are converted to fp16 on their way into LDS)
template <int R, bool FILL, bool PAGED, bool PRESPLIT>
__global__ __launch_bounds__(R * 2) void encode_mfma_kernel(
    const uint16_t* __restrict__ K, const float* __restrict__ W_H, const uint4* __restrict__ planes,
    const int32_t* __restrict__ start, const int32_t* __restrict__ n_new,
    uint32_t* __restrict__ codes, int Hkv, int L_cap, int keys_per_wg,
    int64_t sb, int64_t sh, int64_t sn,
    // fused cache fill (all null otherwise): the keys are read from K_new [B, Hkv, max_new, d] and
    // written to the cache K as they pass through; V_new is copied to V alongside
    const uint16_t* __restrict__ K_new, const uint16_t* __restrict__ V_new,
    uint16_t* __restrict__ K_out, uint16_t* __restrict__ V_out, int max_new,
    // block table of the destination (PAGED instantiation, fused fill only).  Paged pools are
    // [n_pages, Hkv, page_rows, d] / [n_pages, Hkv, page_rows, WD].
    const PageView pv) {
    constexpr int THREADS = R * 2;
    constexpr int WD = R / 32;
    constexpr int STAGE = R < 64 || FILL ? 64 : 128;  // keys per LDS stage
    constexpr int NT = STAGE / 32;                         // 32-key MFMA tiles per stage
    constexpr int ROWS_PER_IT = THREADS / 16;              // rows staged per load instruction
    constexpr int NIT = STAGE / ROWS_PER_IT;               // load instructions per stage and thread
    __shared__ __attribute__((aligned(16))) uint16_t tile[STAGE * HATA_MFMA_PITCH];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m = lane & 31, half = lane >> 5;
    const int h = blockIdx.y, b = blockIdx.z;
    const int first = start[b];
    constexpr bool paged = PAGED;
    int cnt = min(n_new[b], (paged ? min(L_cap, pv.max_blocks << pv.shift) : L_cap) - first);
    if (FILL) cnt = min(cnt, max_new);  // the source holds max_new rows per unit
    const int kb0 = blockIdx.x * keys_per_wg;
    if (first < 0 || kb0 >= cnt) return;
    const int kb1 = min(kb0 + keys_per_wg, cnt);
    const int64_t u = (int64_t)b * Hkv + h;
    const uint16_t* Kb = K + b * sb + h * sh + (int64_t)first * sn;
    uint32_t* cb = codes + (u * L_cap + first) * WD;
    const uint16_t* Ksrc = FILL ? K_new + u * (int64_t)max_new * HATA_D : Kb;
    const uint16_t* Vsrc = FILL ? V_new + u * (int64_t)max_new * HATA_D : nullptr;
    const int64_t src_n = FILL ? HATA_D : sn;
    // paged destination: row (first + key) of sequence b -> row of the pools, in rows of one head
    auto pool_row = [&](int key) -> int64_t {
        const int n = first + key;
        const int p = clampi(pv.table[(int64_t)b * pv.max_blocks + (n >> pv.shift)], 0, pv.n_pages - 1);
        return (((int64_t)p * Hkv + h) << pv.shift) + (n & ((1 << pv.shift) - 1));
    };

    // stage loader: thread -> (row = it * ROWS_PER_IT + tid / 16, 16-byte piece tid % 16)
    const int lrow = tid >> 4, lsub = tid & 15;
    uint4 pre[NIT], vpre[FILL ? NIT : 1];
    int64_t dst[FILL ? NIT : 1];  // where the pieces go in the cache, in elements
    auto load_stage = [&](int k0) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int key = k0 + it * ROWS_PER_IT + lrow;
            if constexpr (PAGED) dst[it] = pool_row(min(key, kb1 - 1)) * HATA_D + lsub * 8;
            else if constexpr (FILL) dst[it] = b * sb + h * sh + (int64_t)(first + key) * sn + lsub * 8;
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            // (rows past the end repeat the last one and are stored nowhere)
            const int64_t o = (int64_t)min(k0 + it * ROWS_PER_IT + lrow, kb1 - 1) * src_n + lsub * 8;
            pre[it] = load_once(Ksrc + o);
            if constexpr (FILL) vpre[it] = load_once(Vsrc + o);
        }
    };
    auto store_stage = [&](int k0) {
        if constexpr (FILL) {
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                if (k0 + it * ROWS_PER_IT + lrow < kb1) {
                    *reinterpret_cast<uint4*>(K_out + dst[it]) = pre[it];
                    *reinterpret_cast<uint4*>(V_out + dst[it]) = vpre[it];
                }
            }
        }
    };
    // the first stage of keys is on its way while the weight fragments arrive
    load_stage(kb0);

    // weight fragments: a[plane][kk] holds W_H[h][kk*16 + 8*half + e][32 w + m], e = 0..7
    bf16x8_t afrag[PRESPLIT ? 1 : 3][PRESPLIT ? 1 : 8];
    f16x8_t afrag16[PRESPLIT ? 2 : 1][PRESPLIT ? 8 : 1];
    if constexpr (PRESPLIT) {
        // prepared once per weight tensor (hata_prepare_weights): 16 coalesced 16-byte loads
        const uint4* src = planes + ((int64_t)(h * (R / 32) + w) * 8 * 2) * 64 + lane;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
#pragma unroll
            for (int p = 0; p < 2; ++p) afrag16[p][kk] = __builtin_bit_cast(f16x8_t, src[(kk * 2 + p) * 64]);
    } else {
        const float* wp = W_H + (int64_t)h * HATA_D * R + w * 32 + m;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            uint32_t hi[4], mid[4], lo[4];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2)
                split_weight_pair(wp[(int64_t)(kk * 16 + 8 * half + 2 * e2) * R],
                                  wp[(int64_t)(kk * 16 + 8 * half + 2 * e2 + 1) * R], hi[e2], mid[e2], lo[e2]);
            afrag[0][kk] = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
            afrag[1][kk] = __builtin_bit_cast(bf16x8_t, make_uint4(mid[0], mid[1], mid[2], mid[3]));
            afrag[2][kk] = __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
        }
    }
    for (int k0 = kb0; k0 < kb1; k0 += STAGE) {
        __syncthreads();  // the previous stage has been consumed
#pragma unroll
        for (int it = 0; it < NIT; ++it)
            *reinterpret_cast<uint4*>(&tile[(it * ROWS_PER_IT + lrow) * HATA_MFMA_PITCH + lsub * 8]) =
                PRESPLIT ? __builtin_bit_cast(uint4, bf16x8_to_f16(pre[it])) : pre[it];
        store_stage(k0);
        __syncthreads();
        if (k0 + STAGE < kb1) load_stage(k0 + STAGE);  // overlaps the MFMAs below

        f32x16_t acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
        // Key fragments come from LDS one channel step ahead: as soon as the planes of a tile have been issued
        // for step kk, the tile's fragment for step kk + 1 is requested into the same registers, so its LDS
        // latency is covered by the MFMAs of the other tiles (nine with four tiles and three planes, two or three in the fill).
        uint4 bfrag[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
            bfrag[t] = *reinterpret_cast<const uint4*>(&tile[(t * 32 + m) * HATA_MFMA_PITCH + 8 * half]);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if constexpr (PRESPLIT) {
#pragma unroll
                    for (int p = 0; p < 2; ++p)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(afrag16[p][kk], __builtin_bit_cast(f16x8_t, bfrag[t]), acc[t], 0, 0, 0);
                } else {
#pragma unroll
                    for (int p = 0; p < 3; ++p)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[p][kk], __builtin_bit_cast(bf16x8_t, bfrag[t]), acc[t], 0, 0, 0);
                }
                if (kk + 1 < 8)
                    bfrag[t] = *reinterpret_cast<const uint4*>(
                        &tile[(t * 32 + m) * HATA_MFMA_PITCH + (kk + 1) * 16 + 8 * half]);
            }
        }
        // sign bits: this lane holds hash columns 8*(i/4) + 4*half + i%4 of key t*32 + m
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            uint32_t word = sign_bits(acc[t]) << (4 * half);
            word |= (uint32_t)__shfl_xor((int)word, 32, 64);
            const int key = k0 + t * 32 + m;
            if (half == 0 && key < kb1) {
                if constexpr (paged) codes[pool_row(key) * WD + w] = word;
                else cb[(int64_t)key * WD + w] = word;
            }
        }
    }
}

// ---- key encode with fp16 weight planes -------------------------------------------------------
// The projection for keys that already lie in a contiguous cache (no fused fill), with weights
// prepared by hata_prepare_weights.  Two things differ from encode_mfma_kernel.
//
// (1) Two fp16 planes instead of three bf16 planes.  With realistic operand values the matrix cores
// of the whole chip sustain about 55 cycles per v_mfma_f32_32x32x16 and SIMD, not 32 (measured with a
// loop of nothing but MFMAs: the rate depends on the values, i.e. on power), and the three-plane kernel's
// stage loop runs at exactly that rate -- so what shortens the kernel is fewer MFMAs.  Per hash-column
// tile (32 columns) the weights are scaled by a power of two S so that max |W S| < 2^14 (signs and
// therefore code bits are unchanged), hi = fp16(W S), lo = fp16(W S - hi): |W S - hi - lo| <= 2^-22 |W S|.
// A bf16 key channel converts to fp16 exactly for 2^-14 <= |x| <= 65504 (eight significant bits);
// smaller values lose at most 2^-25 absolutely, larger ones saturate at 65504.  Every product of two
// fp16 values is exact in the fp32 accumulator.  The projection therefore differs from the exact one by
// at most 2^-22 * sum_c |x_c W_c| (about 5e-6 for the workloads here) plus the fp32 summation error the
// bf16 form has as well: far inside the band of 1e-4 in which code bits may differ from an exact evaluation.
//
// (2) The key rows are staged by the memory pipeline itself: global_load_lds_dwordx4 moves 16 bytes
// per lane from memory straight into LDS (lane l of a wave lands at the instruction's LDS base + 16 l),
// so a stage costs no registers and several stages can be on their way while one is being multiplied.
// A workgroup cycles through NBUF tiles of STAGE keys: in turn s it waits for tile s, passes the
// one barrier of the turn, requests tile s + NBUF - 1 into the buffer that turn s - 1 has just
// finished with, and multiplies tile s.  Two tiles of 128 keys where a workgroup has more than 128, four of 64 for the
// short prompts: half the barriers, and a wave's four independent products cover each other's latency (131072 keys of
// eight heads, r = 256: 133.6 us with four tiles of 64, 125.2 with two of 128, 127.4 with three of 128 and one workgroup per CU;
// 2048 keys, 64 a workgroup: 5.3 and 6.3).
// LDS tile: row r at byte 256 r, unpadded; its 16-byte piece c sits in slot c ^ (r & 15), which makes
// the operand reads (32 rows, one piece index) conflict-free.  A lane of a DMA instruction therefore
// fetches piece slot ^ (row & 15) of its row: 16 lanes still read one whole 256-byte row.
// The rows are converted to fp16 (three VALU instructions per dword) in LDS from r = 128 on, below that as they
// are read.  The code words of a stage go through a small LDS array and leave as 16-byte stores one turn later.

// Fragment order of the fp16 planes: for KV head h, wave w (hash columns 32 w .. 32 w + 31), channel
// step kk and plane p (0 = hi, 1 = lo) the 64 lanes' 16-byte fragments lie one after the other:
//   uint4 index = (((h * (R / 32) + w) * 8 + kk) * 2 + p) * 64 + lane
// grid = (R / 32, Hkv); 64 threads: one wave scales and splits its 32 columns
__global__ __launch_bounds__(64) void split_weights_f16_kernel(const float* __restrict__ W_H, uint4* __restrict__ planes, int R) {
    const int lane = threadIdx.x, w = blockIdx.x, h = blockIdx.y;
    const int m = lane & 31, half = lane >> 5;
    const float* wp = W_H + (int64_t)h * HATA_D * R + w * 32 + m;
    float wv[8][8];
    float mx = 0.f;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            wv[kk][e] = wp[(int64_t)(kk * 16 + 8 * half + e) * R];
            mx = fmaxf(mx, fabsf(wv[kk][e]));  // (fmaxf drops NaN)
        }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    int ex = 14;  // scale 1 for an all-zero or non-finite tile
    if (mx > 0.f && mx < __builtin_inff()) (void)frexpf(mx, &ex);  // mx = f 2^ex, 0.5 <= f < 1
    const int sh = 14 - ex;                                        // max |W| 2^sh < 2^14
    uint4* dst = planes + ((int64_t)(h * (R / 32) + w) * 8 * 2) * 64 + lane;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        f16x8_t hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float ws = ldexpf(wv[kk][e], sh);
            hi[e] = (_Float16)ws;                 // round to nearest even
            lo[e] = (_Float16)(ws - (float)hi[e]);  // (the difference is exact in fp32)
        }
        dst[(kk * 2 + 0) * 64] = __builtin_bit_cast(uint4, hi);
        dst[(kk * 2 + 1) * 64] = __builtin_bit_cast(uint4, lo);
    }
}

template <int R, int STAGE>
__global__ __launch_bounds__(R * 2) void encode_dma_kernel(
    const uint16_t* __restrict__ K, const uint4* __restrict__ planes,
    const int32_t* __restrict__ start, const int32_t* __restrict__ n_new, uint32_t* __restrict__ codes,
    int Hkv, int L_cap, int keys_per_wg, int64_t sb, int64_t sh, int64_t sn) {
    constexpr int WAVES = R / 32, WD = R / 32;
    constexpr int NBUF = 256 / STAGE;              // 64 KB of tiles
    constexpr int NT = STAGE / 32;                 // 32-key MFMA tiles per stage
    constexpr int INSTR = STAGE / (WAVES * 4);     // DMA instructions per wave and stage (4 rows each)
    static_assert(INSTR >= 1 && INSTR * WAVES * 4 == STAGE, "a stage is a whole number of DMA instructions per wave");
    __shared__ __attribute__((aligned(16))) uint4 tile[NBUF][STAGE * 16];
    __shared__ __attribute__((aligned(16))) uint32_t cbuf[2][STAGE * WD];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m = lane & 31, half = lane >> 5;
    const int h = blockIdx.y, b = blockIdx.z;
    const int first = start[b];
    const int cnt = min(n_new[b], L_cap - first);
    const int kb0 = blockIdx.x * keys_per_wg;
    if (first < 0 || kb0 >= cnt) return;
    const int kb1 = min(kb0 + keys_per_wg, cnt);
    const int64_t u = (int64_t)b * Hkv + h;
    const uint16_t* Kb = K + b * sb + h * sh + (int64_t)first * sn;
    uint32_t* cb = codes + (u * L_cap + first) * WD;
    const int n_stages = (kb1 - kb0 + STAGE - 1) / STAGE;

    // rows past the end of the range are fetched from the range's last row (valid memory; their code
    // words are never stored)
    const int drow = lane >> 4, dslot = lane & 15;
    auto request = [&](int s) {
        const int k0 = kb0 + s * STAGE;
        uint4* dst = &tile[s % NBUF][0];
#pragma unroll
        for (int it = 0; it < INSTR; ++it) {
            const int r0 = (it * WAVES + w) * 4;
            const int row = r0 + drow;
            const int key = min(k0 + row, kb1 - 1);
            const uint16_t* g = Kb + (int64_t)key * sn + ((dslot ^ (row & 15)) * 8);
            // (written as an instruction: given the compiler's builtin for it, every later LDS read is
            // made to wait for ALL requests outstanding, which is the one thing this kernel must not do;
            // the waits are the explicit ones in the stage loop)
            const uint32_t lds_base = __builtin_amdgcn_readfirstlane(
                (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(dst + r0 * 16));
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                         :: "s"(lds_base), "v"(g) : "memory", "m0");
        }
    };
    // weight fragments first (they are needed for as long as the kernel runs), then the first tiles
    f16x8_t afrag[2][8];
    {
        const uint4* src = planes + ((int64_t)(h * (R / 32) + w) * 8 * 2) * 64 + lane;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
#pragma unroll
            for (int p = 0; p < 2; ++p) afrag[p][kk] = __builtin_bit_cast(f16x8_t, src[(kk * 2 + p) * 64]);
    }
#pragma unroll
    for (int s = 0; s < NBUF - 1; ++s)
        if (s < n_stages) request(s);
    // the weight fragments are there before the loop starts (said explicitly, or the compiler guards
    // their every use inside the loop with a count of outstanding loads that fits the first turn only)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)

    // 16-byte pieces of the previous stage's code words that this thread stores (none for most threads)
    constexpr int CODE_VEC = STAGE * WD / 4;
    static_assert(WD < 4 || CODE_VEC <= R * 2, "a thread stores one piece at most");
    auto flush_codes = [&](int s) {  // code words of stage s, staged in cbuf[s & 1]
        const int k0 = kb0 + s * STAGE;
        if constexpr (WD >= 4) {  // (a key's code is 16 bytes or more: every piece is aligned)
            if (tid < CODE_VEC && k0 + (tid * 4) / WD < kb1)
                reinterpret_cast<uint4*>(cb + (int64_t)k0 * WD)[tid] = reinterpret_cast<const uint4*>(&cbuf[s & 1][0])[tid];
        } else {
            for (int i = tid; i < STAGE * WD; i += R * 2)
                if (k0 + i / WD < kb1) cb[(int64_t)k0 * WD + i] = cbuf[s & 1][i];
        }
    };
    // At r >= 128 a tile is converted in place, each wave its own requests: four or eight waves would
    // otherwise each convert all of it (r = 256, 131072 keys of eight heads: 146.2 -> 131.6 us; at r = 64
    // converting what is read is the faster one, 56.3 against 59.2).
    constexpr bool ONCE = R >= 128;
    // This wave's part of tile s.  It has landed once at most the requests made after it are outstanding: those of
    // the NBUF - 2 tiles that follow (stores of code words, if any, only make this wait longer).
    auto landed = [&](int s) {
        if (s + NBUF - 2 < n_stages) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NBUF - 2) * INSTR) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    // the 16-byte pieces of tile s that this lane requested (a lane's piece lands at the instruction's base + 16 lane)
    auto convert = [&](int s) {
        uint4* p = &tile[s % NBUF][w * 64 + lane];
#pragma unroll
        for (int it = 0; it < INSTR; ++it)
            p[it * WAVES * 64] = __builtin_bit_cast(uint4, bf16x8_to_f16(p[it * WAVES * 64]));
    };
    if constexpr (ONCE) {
        asm volatile("" ::: "memory");
        convert(0);
    }
    for (int s = 0; s < n_stages; ++s) {
        if constexpr (!ONCE) landed(s);
        __syncthreads();  // every wave's part of tile s is there (and converted); everybody is done with tile s - 1
        if (s + NBUF - 1 < n_stages) request(s + NBUF - 1);
        if (s > 0) flush_codes(s - 1);
        const uint4* tl = &tile[s % NBUF][0];
        f32x16_t acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
        // Key fragments are read from LDS two channel steps ahead and, where they are bf16 still, converted one
        // step ahead, so that neither the LDS latency nor the conversion stands in front of an MFMA (the
        // scheduler is told to keep the steps apart: left alone it moves each read down to its first use)
        const int at0 = m * 16 + (half ^ (m & 15));
        auto piece = [&](int kk, int t) { return tl[t * 512 + (at0 ^ (2 * kk))]; };
        auto operand = [](const uint4& v) { return ONCE ? __builtin_bit_cast(f16x8_t, v) : bf16x8_to_f16(v); };
        uint4 raw[NT];
        f16x8_t bcur[NT], bnext[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) raw[t] = piece(0, t);
#pragma unroll
        for (int t = 0; t < NT; ++t) bcur[t] = operand(raw[t]);
#pragma unroll
        for (int t = 0; t < NT; ++t) raw[t] = piece(1, t);
        __builtin_amdgcn_s_setprio(1);  // a wave that multiplies goes before one that converts or packs (1 %)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            __builtin_amdgcn_sched_barrier(0);
            if (kk + 1 < 8) {
#pragma unroll
                for (int t = 0; t < NT; ++t) bnext[t] = operand(raw[t]);
            }
            if (kk + 2 < 8) {
#pragma unroll
                for (int t = 0; t < NT; ++t) raw[t] = piece(kk + 2, t);
            }
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(afrag[p][kk], bcur[t], acc[t], 0, 0, 0);
            if constexpr (!ONCE) {
                // one MFMA, then a quarter of the step's conversions in its shadow
#pragma unroll
                for (int q = 0; q < 2 * NT; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);           // MFMA
                    __builtin_amdgcn_sched_group_barrier(0x002, 12 / 2, 0);      // VALU
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < NT; ++t) bcur[t] = bnext[t];
        }
        __builtin_amdgcn_s_setprio(0);
        if constexpr (ONCE) {
            if (s + 1 < n_stages) {  // in the shadow of the last MFMAs
                landed(s + 1);
                convert(s + 1);
            }
        }
        // sign bits: this lane holds hash columns 8*(i/4) + 4*half + i%4 of key t*32 + m
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            uint32_t word = sign_bits(acc[t]) << (4 * half);
            word |= (uint32_t)__shfl_xor((int)word, 32, 64);
            if (half == 0) cbuf[s & 1][(t * 32 + m) * WD + w] = word;
        }
    }
    __syncthreads();
    flush_codes(n_stages - 1);
}

hipError_t launch_encode_vectors(const hata_ctx* c, const void* q, uint32_t* qcodes,
                                 const void* K, const int32_t* start, const int32_t* n_new,
                                 int max_new, int from_seq_len, uint32_t* codes,
                                 const float* W_H, int B, hipStream_t s) {
    const hata_config& f = c->cfg;
    if (!q && !K) return hipSuccess;
    const bool one = (q ? c->G : 0) + (K ? (from_seq_len ? 1 : max_new) : 0) == 1;
#define HATA_LAUNCH_FEW(COLS)                                                                                       \
    hipLaunchKernelGGL((one ? encode_few_kernel<COLS, true> : encode_few_kernel<COLS, false>), dim3(f.r / COLS, B * f.Hkv), dim3(256), 0, s, (const uint16_t*)q, \
                       qcodes, (const uint16_t*)K, start, n_new, max_new, from_seq_len, codes, W_H, f.Hq, f.Hkv,    \
                       c->G, f.r, f.L_cap, f.kv_stride_b, f.kv_stride_h, f.kv_stride_n)
    if (f.r % 64 == 0) HATA_LAUNCH_FEW(64);
    else HATA_LAUNCH_FEW(32);
#undef HATA_LAUNCH_FEW
    return hipGetLastError();
}

hipError_t launch_encode_bulk(const hata_ctx* c, const void* K, const float* W_H,
                              const int32_t* start, const int32_t* n_new, int B, int max_new,
                              uint32_t* codes, hipStream_t s, const void* K_new, const void* V_new,
                              void* K_out, void* V_out, const PageView* pages) {
    const hata_config& f = c->cfg;
    const PageView pv = pages ? *pages : PageView{nullptr, 0, 0, 0};
    if (pages && !K_new) return hipErrorNotSupported;  // the block table addresses the fused fill only
    if (max_new <= 0 || B <= 0) return hipSuccess;
    const uint16_t* kn = (const uint16_t*)K_new;
    const uint16_t* vn = (const uint16_t*)V_new;
    uint16_t* ko = (uint16_t*)K_out;
    uint16_t* vo = (uint16_t*)V_out;
    if (f.r == 32 || f.r == 64 || f.r == 128 || f.r == 256) {
        // the weight planes prepared for exactly this weight tensor, if any (hata_prepare_weights)
        const uint4* planes = (c->prepared_W_H == W_H && c->wplanes) ? (const uint4*)c->wplanes : nullptr;
        // Keys per workgroup, 64 to 4096.  Every workgroup fetches the head's weight planes, so no more of them than
        // two per CU; a short prompt then has few keys a workgroup, because one after the other they take 2.6 us
        // per stage (2048 keys, eight heads, r = 128: 512 / 128 / 64 keys a workgroup 13.0 / 5.1 / 4.4 us).  The fill
        // takes up to eight per CU where the weights are small next to its rows: it has more to
        // request than two can have on the way (paged fill of 8011 tokens, r = 128: 128 / 512 keys
        // 35.0 / 38.1 us; r = 256, 2 x 32768: 128 / 1024 keys 126 / 93 us).  Weights split by the
        // workgroup itself cost more than a second stage: 128 at least (8192 keys, r = 128: 64 / 128 keys
        // 21.6 / 12.5 us), and with one or two waves a workgroup up to four of them per CU (32768 keys, r = 64:
        // 256 / 512 keys 21.1 / 25.3 us).
        const int64_t most = kn && planes && f.r <= 128 ? 2048 : !planes && f.r <= 64 ? 1024 : 512;
        auto wgs = [&](int k) { return (int64_t)((max_new + k - 1) / k) * f.Hkv * B; };
        int kpw = 4096;
        while (kpw > 128 && wgs(kpw) < most) kpw >>= 1;
        if (planes && wgs(kpw) < 512) kpw = 64;
        const dim3 grid((max_new + kpw - 1) / kpw, f.Hkv, B);
        if (!kn && !pages && planes) {
            // keys already in a contiguous cache, weights prepared: the kernel that stages with LDS-direct loads
            const uint4* p16 = planes;
#define HATA_LAUNCH_DMA(R_)                                                                                          \
    hipLaunchKernelGGL((kpw > 128 ? encode_dma_kernel<R_, 128> : encode_dma_kernel<R_, 64>), grid, dim3(R_ * 2), 0, s, \
                       (const uint16_t*)K, p16, start, n_new, codes, f.Hkv, f.L_cap, kpw, f.kv_stride_b,             \
                       f.kv_stride_h, f.kv_stride_n)
            if (f.r == 32) HATA_LAUNCH_DMA(32);
            else if (f.r == 64) HATA_LAUNCH_DMA(64);
            else if (f.r == 128) HATA_LAUNCH_DMA(128);
            else HATA_LAUNCH_DMA(256);
#undef HATA_LAUNCH_DMA
            return hipGetLastError();
        }
#define HATA_LAUNCH_MFMA(R_, F_, P_, S_)                                                                       \
    hipLaunchKernelGGL((encode_mfma_kernel<R_, F_, P_, S_>), grid, dim3(R_ * 2), 0, s, (const uint16_t*)K, W_H, planes, \
                       start, n_new, codes, f.Hkv, f.L_cap, kpw, f.kv_stride_b, f.kv_stride_h, f.kv_stride_n, kn, vn,   \
                       ko, vo, max_new, pv)
#define HATA_LAUNCH_WIDTH(F_, P_, S_)                          \
    do {                                                       \
        if (f.r == 32) HATA_LAUNCH_MFMA(32, F_, P_, S_);       \
        else if (f.r == 64) HATA_LAUNCH_MFMA(64, F_, P_, S_);  \
        else if (f.r == 128) HATA_LAUNCH_MFMA(128, F_, P_, S_); \
        else HATA_LAUNCH_MFMA(256, F_, P_, S_);                \
    } while (0)
        if (!kn) HATA_LAUNCH_WIDTH(false, false, false);
        else if (pages && planes) HATA_LAUNCH_WIDTH(true, true, true);
        else if (pages) HATA_LAUNCH_WIDTH(true, true, false);
        else if (planes) HATA_LAUNCH_WIDTH(true, false, true);
        else HATA_LAUNCH_WIDTH(true, false, false);
#undef HATA_LAUNCH_WIDTH
#undef HATA_LAUNCH_MFMA
        return hipGetLastError();
    }
    if (kn) return hipErrorNotSupported;  // the fused cache fill exists for the MFMA widths only
    const int tiles = (max_new + 63) / 64;
    hipLaunchKernelGGL(encode_bulk_kernel, dim3(tiles, f.Hkv, B), dim3(256), 0, s,
                       (const uint16_t*)K, W_H, start, n_new, codes, f.Hkv, f.r, c->Wd, f.L_cap,
                       f.kv_stride_b, f.kv_stride_h, f.kv_stride_n);
    return hipGetLastError();
}

// Split of the fp32 hash weights into two scaled fp16 planes in the operand-fragment order of the key encoders
hipError_t launch_split_weights(const hata_ctx* c, const float* W_H, hipStream_t s) {
    const hata_config& f = c->cfg;
    hipLaunchKernelGGL(split_weights_f16_kernel, dim3(f.r / 32, f.Hkv), dim3(64), 0, s, W_H, (uint4*)c->wplanes, f.r);
    return hipGetLastError();
}

}  // namespace hata
