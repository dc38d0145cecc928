// Decode attention over the whole cache (Eq. 1 of the paper; the dense layers of Alg. 1 and the baseline that the
// method is compared with).
//
// Bound by the HBM stream: every K and V row is read once for all query heads of its group.
//   - A workgroup of eight waves owns a run of 16-row tiles; the launch is sized to one workgroup per CU, so that
//     the tail of the stream and the number of partial results to merge are both small, and dealt out by the
//     sequences' lengths (dense_share), so that it stays even when one of them is long and the others are not.
//   - Every wave requests its tiles with direct loads into a wave-private LDS ring (no registers, no barriers: the
//     only waits in the loop are the ones for a tile's own K and V), whole 256-byte rows per 16 lanes.  The 16-byte
//     pieces of row r are stored in the order piece ^ swizzle(r), which makes both kinds of reads below free
//     of bank conflicts.
//   - The contractions are those of attn_rows_mfma (hata_attn_core.h), heads padded to 16, with the softmax weights as
//     two bf16 terms -- for the groups whose sparse attention takes them that way too (tiles of four heads or
//     more).  The other groups' weights stay fp32, and products with them are as in plain fp32 also where a value is
//     infinite: with one or two heads on the vector ALU (the padding repeats the heads, so a lane has the weights of
//     its rows), else in the fp32 matrix instructions, 32 a tile instead of 8 (two heads that way,
//     16 KV heads of 32768 rows: 52 us; on the vector ALU 45).
// Measured at B = 1, 8 KV heads, 32768 rows (134 MB), groups of 4 and 8 heads: 25.7 and 29.2 us; four waves per
// workgroup with loads through registers and 64 partial results per unit took 36.8 and 48.7.  B = 4, 65536 rows,
// groups of 8 (1.07 GB): 167 us, 6.4 TB/s (209).
#include <algorithm>
#include "hata_device.h"
#include "hata_internal.h"
#include "hata_attn_core.h"

namespace hata {

// (measured at B = 1, 32768 rows, groups of 4, loads not yet marked non-temporal: 8 waves x 2 tiles 29.0 us; 4 x 4
// 32.2; 6 x 3 31.3; two workgroups of 4 x 2 per CU 33.4)
#define DENSE_WAVES 8
#define DENSE_RING 2           // tiles in flight per wave
#define DENSE_TILE_BYTES 8192  // 16 rows of K, 16 rows of V
#define DENSE_RUN 4            // tiles (of a wave) summed in a row where the weights stay fp32
#define DENSE_MAX_RUNS 256     // of a unit (four partial results per lane in the merge)
#define DENSE_BATCH 16         // partial results in flight per thread in the merge

struct DenseArgs {
    const uint16_t *q, *K, *V;
    const int32_t* seq_len;
    float* partials;
    uint32_t* counter;
    int counter_stride;
    uint16_t* out;
    float* out_f32;
    int Hq, Hkv, G, B, L_cap;
    int64_t sb, sh, sn;
    float scale_log2;
};

// two heads in the even and odd lanes: the neighbour's value
__device__ __forceinline__ float other_head(float v) { return HATA_DPP(v, 0xB1); }  // quad_perm [1,0,3,2]

__device__ __forceinline__ int dense_swizzle(int r) { return ((r << 1) | (r >> 3)) & 15; }

template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// waits until at most FIRST requests of this tile and all of the next one, if there is one, are outstanding
template <int FIRST>
__device__ __forceinline__ void wait_tile(int tiles_after) {
    static_assert(DENSE_RING == 2, "one more tile in flight");
    if (tiles_after >= 1) wait_vm<FIRST + 8>();
    else wait_vm<FIRST>();
}

// What a workgroup of the launch works on: split `split` of the ns runs that unit (b, h) is cut into, `first` the
// workgroup that has its first one
struct DenseShare { int b, h, L, split, ns, first; };

// The launch's workgroups (at least one per unit) in proportion to the sequences' lengths: the shortest run length, from
// an even share of all tiles and a tile per wave up in steps of an eighth, at which the units' runs are no more than
// the workgroups.  (Cut by the longest sequence there could be, 16 sequences of which one has 32768 rows and the others
// 2048 took 167 us, this takes 50; 8 KV heads.)  Every wave of every workgroup computes the same; false: nothing left for this one.
__device__ __forceinline__ bool dense_share(const int32_t* __restrict__ seq_len, int B, int Hkv, int L_cap, DenseShare& d) {
    if (B == 1) {  // nothing to weigh up: which head this is does not wait for the length
        const int per = gridDim.x;
        d.b = 0;
        d.h = blockIdx.y;
        d.split = blockIdx.x;
        d.first = d.h * per;
        d.L = clampi(seq_len[0], 0, L_cap);
        d.ns = clampi(((d.L + 15) / 16 + DENSE_WAVES - 1) / DENSE_WAVES, 1, per);
        return d.split < d.ns;
    }
    const int lane = threadIdx.x & 63, wg = blockIdx.x, wgs = gridDim.x;
    auto length = [&](int b) { return b < B ? clampi(seq_len[b], 0, L_cap) : -1; };
    const int own = length(lane);  // the only round trip for up to 64 sequences
    auto of = [&](int b0) { return b0 == 0 ? own : length(b0 + lane); };
    // (a sequence without rows: one workgroup writes zeros)
    auto tiles = [](int L) { return L >= 0 ? (max(L, 1) + 15) / 16 : 0; };
    float all = 0.f;
    for (int b0 = 0; b0 < B; b0 += 64) all += wave_sum64((float)tiles(of(b0)));
    int run = max(DENSE_WAVES, (int)ceilf(all * (float)Hkv * __builtin_amdgcn_rcpf((float)wgs)));
    // (the quotients are exact below 2^20, and a cache has fewer tiles)
    auto quotient = [](int x, int y) { return (int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)y)); };
    auto runs = [&](int L) { return (uint32_t)min(quotient(tiles(L) + run - 1, run), DENSE_MAX_RUNS); };
    uint32_t upto;  // runs of the sequences up to this lane's, of the last 64 looked at
    for (;; run += max(1, run >> 3)) {  // (ends at the cache's tiles at the latest: one run a unit)
        uint32_t n = 0;
        for (int b0 = 0; b0 < B; b0 += 64) {
            upto = wave_incl_scan(runs(of(b0)));
            n += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        }
        if (n * (uint32_t)Hkv <= (uint32_t)wgs || run >= tiles(L_cap)) break;
    }
    int before = 0;
    for (int b0 = 0; b0 < B; b0 += 64) {
        const int L = of(b0), n = (int)runs(L);
        if (B > 64) upto = wave_incl_scan((uint32_t)n);
        const unsigned long long past = __builtin_amdgcn_ballot_w64(before + Hkv * (int)upto > wg);
        if (past) {
            const int l = __ffsll(past) - 1;
            d.b = b0 + l;
            d.L = __builtin_amdgcn_readlane(L, l);
            d.ns = __builtin_amdgcn_readlane(n, l);
            const int in_seq = wg - before - Hkv * (__builtin_amdgcn_readlane((int)upto, l) - d.ns);
            d.h = __builtin_amdgcn_readfirstlane(quotient(in_seq, d.ns));
            d.split = in_seq - d.h * d.ns;
            d.first = wg - d.split;
            return true;
        }
        before += Hkv * __builtin_amdgcn_readlane((int)upto, 63);
    }
    return false;
}

enum DenseForm { DENSE_BF16X2, DENSE_FP32_ONE_HEAD, DENSE_FP32_TWO_HEADS, DENSE_FP32 };
template <DenseForm FORM>
__global__ __launch_bounds__(DENSE_WAVES * 64) void dense_kernel(const DenseArgs a) {
    // ring[wave][DENSE_RING][DENSE_TILE_BYTES]; afterwards the waves' states, the merge weights and sums
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ float s_m[DENSE_WAVES][16], s_l[DENSE_WAVES][16];
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kg = lane >> 4;
    DenseShare d;
    if (!dense_share(a.seq_len, a.B, a.Hkv, a.L_cap, d)) return;
    const int split = d.split, ns = d.ns, h = d.h, b = d.b, L = d.L, G = a.G;
    const int64_t u = (int64_t)b * a.Hkv + h, hq0 = (int64_t)b * a.Hq + (int64_t)h * G;
    uint16_t* outp = a.out + hq0 * HATA_D;
    float* outp32 = a.out_f32 ? a.out_f32 + hq0 * HATA_D : nullptr;
    uint4 qb[4];
    {
        const uint16_t* q0 = a.q + (hq0 + (FORM == DENSE_FP32_TWO_HEADS ? n & 1 : min(n, G - 1))) * HATA_D + 8 * kg;
#pragma unroll
        for (int s = 0; s < 4; ++s) qb[s] = *reinterpret_cast<const uint4*>(q0 + 32 * s);
    }
    if (L == 0) {  // no row at all
        for (int i = tid; i < G * HATA_D; i += DENSE_WAVES * 64) {
            outp[i] = 0;
            if (outp32) outp32[i] = 0.f;
        }
        return;
    }
    const int tiles = (L + 15) / 16;  // in even runs
    const int t_begin = (int)((int64_t)tiles * split / ns), t_end = (int)((int64_t)tiles * (split + 1) / ns);
    const int mine = max(0, (t_end - t_begin - wave + DENSE_WAVES - 1) / DENSE_WAVES);  // tiles t_begin + wave + 8 j

    const uint16_t* Kb = a.K + b * a.sb + h * a.sh;
    const uint16_t* Vb = a.V + b * a.sb + h * a.sh;
    char* ring = smem + wave * (DENSE_RING * DENSE_TILE_BYTES);
    const uint32_t ring_lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)ring);
    // request: lane l of instruction i fetches piece (l % 16) ^ swizzle(row) of row 4 i + l / 16
    int64_t off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) off[i] = (4 * i + kg) * a.sn + (n ^ dense_swizzle(4 * i + kg)) * 8;
    auto request = [&](int j) {
        const int row0 = (t_begin + wave + DENSE_WAVES * j) * 16;
        const uint16_t* kt = Kb + row0 * a.sn;
        const uint16_t* vt = Vb + row0 * a.sn;
        const uint32_t dst = ring_lds + (uint32_t)(j % DENSE_RING) * DENSE_TILE_BYTES;
        const int last = L - 1 - row0;  // rows past the end repeat the last one
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int64_t o = off[i];
            if (last < 15 && 4 * i + kg > last) o += (int64_t)(last - 4 * i - kg) * a.sn;
            // (written as instructions: behind the compiler's builtin for it, every LDS read waits for all
            // requests outstanding.  nt: the rows are read once, and marked so they stream at 6.1 instead of
            // 5.35 TB/s, 131072 rows)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt"
                         ::"s"(dst + i * 1024), "v"(kt + o) : "memory", "m0");
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int64_t o = off[i];
            if (last < 15 && 4 * i + kg > last) o += (int64_t)(last - 4 * i - kg) * a.sn;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt"
                         ::"s"(dst + 4096 + i * 1024), "v"(vt + o) : "memory", "m0");
        }
    };
    float m_run = HATA_NEG_INF, l_run = 0.f;
    f32x4_t acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    // fp32 forms: sums of DENSE_RUN tiles are added up here, so that no sum is a long chain of small addends (a long chain
    // doubled the error against fp64 at 32768 rows: 4.2e-7 against 2.0e-7).  On the vector ALU acc[2 i] and acc[2 i + 1]
    // are channels 8 n .. 8 n + 7 over rows 4 kg .. 4 kg + 3, of head n % VH (i = 0) and of the other one (i = 1).
    constexpr bool FP32W = FORM != DENSE_BF16X2;
    constexpr int VH = FORM == DENSE_FP32_ONE_HEAD ? 1 : FORM == DENSE_FP32_TWO_HEADS ? 2 : 0;  // heads on the vector ALU
    constexpr int NT = VH ? 2 * VH : FP32W ? 8 : 1;
    [[maybe_unused]] f32x4_t total[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) total[c] = acc[c];
    // K operand: row n, piece 4 s + kg; V operand: row 4 kg + n / 4, channels 16 c + 4 (n % 4), piece 2 c + (n % 4) / 2
    const uint32_t k_at = n * 256 + ((kg ^ dense_swizzle(n)) << 4);
    const int vr = 4 * kg + n / 4;
    const uint32_t v_at = 4096 + vr * 256 + ((((n & 3) >> 1) ^ dense_swizzle(vr)) << 4) + (n & 1) * 8;
    auto compute = [&](int j) {
        const char* t = ring + (j % DENSE_RING) * DENSE_TILE_BYTES;
        const int after = mine - 1 - j;
        const int left = min(L - (t_begin + wave + DENSE_WAVES * j) * 16, 16);
        wait_tile<4>(after);
        // (fp32 forms: four sums of 32 channels instead of one of 128, for the same reason as above)
        f32x4_t sacc, part[4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            part[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(t + (k_at ^ (s << 6)))),
                __builtin_bit_cast(bf16x8_t, qb[s]), s == 0 || FP32W ? (f32x4_t){0.f, 0.f, 0.f, 0.f} : part[s - (s > 0)], 0, 0, 0);
        sacc = FP32W ? (part[0] + part[1]) + (part[2] + part[3]) : part[3];
        // online softmax of head n over the rows 4 kg .. 4 kg + 3 this lane holds
        float sv[4], m_tile = HATA_NEG_INF;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            sv[r] = 4 * kg + r < left ? sacc[r] * a.scale_log2 : HATA_NEG_INF;
            m_tile = fmaxf(m_tile, sv[r]);
        }
        m_tile = rows_max4(m_tile);
        const float m_new = fmaxf(m_run, m_tile);
        const float alpha = (m_new == HATA_NEG_INF) ? 1.f : fast_exp2(m_run - m_new);
        float p[4], psum = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = (sv[r] == HATA_NEG_INF) ? 0.f : fast_exp2(sv[r] - m_new);
            psum += p[r];
        }
        l_run = fmaf(l_run, alpha, psum);
        m_run = m_new;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0ull) {
#pragma unroll
            for (int c = 0; c < (FP32W ? NT : 8); ++c) {
                const float f = VH && c >= 2 ? other_head(alpha) : alpha;
                acc[c] *= f;
                if constexpr (FP32W) total[c] *= f;
            }
        }
        // P as two bf16 terms: hi = p truncated to bf16, lo = (p - hi) truncated to bf16
        [[maybe_unused]] uint4 pb;
        if constexpr (!FP32W) {
            uint32_t hb[4], lb[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                hb[r] = __float_as_uint(p[r]) & 0xffff0000u;
                lb[r] = __float_as_uint(p[r] - __uint_as_float(hb[r]));
            }
            pb = make_uint4((hb[0] >> 16) | hb[1], (hb[2] >> 16) | hb[3],
                            (lb[0] >> 16) | (lb[1] & 0xffff0000u), (lb[2] >> 16) | (lb[3] & 0xffff0000u));
        }
        wait_tile<0>(after);
        uint2 v[8];  // vector ALU: 8 channels of rows 4 kg .. 4 kg + 3, else four rows of channel 16 c + n
        if constexpr (VH > 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * kg + r;
                const uint4 x = *reinterpret_cast<const uint4*>(t + 4096 + row * 256 + ((n ^ dense_swizzle(row)) << 4));
                v[2 * r] = make_uint2(x.x, x.y);
                v[2 * r + 1] = make_uint2(x.z, x.w);
            }
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const s16x4_t av = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4_t*)const_cast<char*>(t + (v_at ^ (c << 5))));
                v[c] = __builtin_bit_cast(uint2, av);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // every read of this slot has returned
        if (left < 16) {  // the copies of the last row past the end: p = 0, and 0 for infinite values
            const int keep = clampi(left - 4 * kg, 0, 4);  // rows of this lane
            const uint32_t lo = keep >= 2 ? 0xffffffffu : keep == 1 ? 0xffffu : 0u;
            const uint32_t hi = keep >= 4 ? 0xffffffffu : keep == 3 ? 0xffffu : 0u;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                if constexpr (VH > 0) {
                    if (c / 2 >= keep) v[c] = make_uint2(0, 0);
                } else {
                    v[c].x &= lo; v[c].y &= hi;
                }
            }
        }
        if (after >= DENSE_RING) request(j + DENSE_RING);
        if constexpr (FP32W) {
            if constexpr (VH > 0) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c < NT; ++c) {
                        const uint2 w = v[2 * r + (c & 1)];
                        const float f = c >= 2 ? other_head(p[r]) : p[r];
                        acc[c][0] = fmaf(f, bf16_lo(w.x), acc[c][0]);
                        acc[c][1] = fmaf(f, bf16_hi(w.x), acc[c][1]);
                        acc[c][2] = fmaf(f, bf16_lo(w.y), acc[c][2]);
                        acc[c][3] = fmaf(f, bf16_hi(w.y), acc[c][3]);
                    }
            } else {
                // rows 4 kg + r in one product: lane (n, kg) has V of channel 16 c + n and the weight of head n
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        const uint32_t w = r < 2 ? v[c].x : v[c].y;
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32((r & 1) ? bf16_hi(w) : bf16_lo(w), p[r], acc[c], 0, 0, 0);
                    }
            }
            if (j % DENSE_RUN == DENSE_RUN - 1 || after == 0) {
#pragma unroll
                for (int c = 0; c < NT; ++c) {
                    total[c] += acc[c];
                    acc[c] = after == 0 ? total[c] : (f32x4_t){0.f, 0.f, 0.f, 0.f};
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, make_uint4(v[c].x, v[c].y, v[c].x, v[c].y)),
                                                                 __builtin_bit_cast(bf16x8_t, pb), acc[c], 0, 0, 0);
        }
    };
    for (int j = 0; j < min(mine, DENSE_RING); ++j) request(j);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (!VH && n >= G) qb[s] = make_uint4(0, 0, 0, 0);
        // (used here, so that the wait for these loads is not in the loop)
        asm volatile("" : "+v"(qb[s].x), "+v"(qb[s].y), "+v"(qb[s].z), "+v"(qb[s].w));
    }
    for (int j = 0; j < mine; ++j) compute(j);

    // ---- the eight states of the workgroup ----
    __syncthreads();  // the ring is no longer read
    float* s_acc = reinterpret_cast<float*>(smem);  // [DENSE_WAVES][G][HATA_D + 4]
    l_run = rows_sum4(l_run);
    if constexpr (VH > 0) {
#pragma unroll
        for (int i = 0; i < 4 * NT; ++i) acc[i / 4][i % 4] = rows_sum4(acc[i / 4][i % 4]);
        if (kg == 0) {
            if (n < VH) { s_m[wave][n] = m_run; s_l[wave][n] = l_run; }
#pragma unroll
            for (int c = 0; c < NT; ++c)
                *reinterpret_cast<float4*>(&s_acc[(wave * VH + (n + c / 2) % VH) * (HATA_D + 4) + 8 * n + 4 * (c & 1)]) =
                    make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
        }
    } else if (n < G) {
        if (kg == 0) { s_m[wave][n] = m_run; s_l[wave][n] = l_run; }
#pragma unroll
        for (int c = 0; c < 8; ++c)  // acc[c][r] = O[head n][channel 16 c + 4 kg + r]
            *reinterpret_cast<float4*>(&s_acc[(wave * G + n) * (HATA_D + 4) + 16 * c + 4 * kg]) =
                make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
    }
    __syncthreads();
    const int64_t head_stride = (int64_t)ns * HATA_PSTRIDE;
    float* part0 = a.partials + (int64_t)d.first * G * HATA_PSTRIDE;  // the unit's: [G][ns]
    for (int i = tid; i < G * HATA_D; i += DENSE_WAVES * 64) {
        const int g = i / HATA_D, ch = i % HATA_D;
        float M = s_m[0][g];
#pragma unroll
        for (int w = 1; w < DENSE_WAVES; ++w) M = fmaxf(M, s_m[w][g]);
        float av = 0.f, l = 0.f;
#pragma unroll
        for (int w = 0; w < DENSE_WAVES; ++w) {
            const float f = M == HATA_NEG_INF ? 0.f : fast_exp2(s_m[w][g] - M);
            av = fmaf(f, s_acc[(w * G + g) * (HATA_D + 4) + ch], av);
            l = fmaf(f, s_l[w][g], l);
        }
        if (ns == 1) {
            const float o = l > 0.f ? av / l : 0.f;
            outp[i] = (uint16_t)f32_to_bf16(o);
            if (outp32) outp32[i] = o;
        } else {
            float* pp = part0 + g * head_stride + split * HATA_PSTRIDE;
            st_dev(pp + 2 + ch, av);
            if (ch == 0) { st_dev(pp, M); st_dev(pp + 1, l); }
        }
    }
    if (ns == 1) return;
    // ---- the last workgroup of the unit merges (partials: write-through stores, device-coherent loads) ----
    wait_stores();
    __syncthreads();
    if (tid == 0) {
        uint32_t* cnt = a.counter + u * a.counter_stride;
        const int last = atomicAdd(cnt, 1u) == (uint32_t)(ns - 1);
        if (last) *cnt = 0;
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    // thread: slices part, part + parts, ... of one head's channel pair; the first batch of loads before the weights
    float* s_w = reinterpret_cast<float*>(smem);                    // [G][ns] normalised weights
    float2* s_sum = reinterpret_cast<float2*>(s_w + ((G * ns + 3) & ~3));  // [parts][G * 64]
    const int items = G * (HATA_D / 2);
    const int parts = max(1, DENSE_WAVES * 64 / items);
    auto address = [&](int i) {
        return part0 + (i / (HATA_D / 2)) * head_stride + 2 + 2 * (i % (HATA_D / 2));
    };
    for (int i0 = 0; i0 < items; i0 += DENSE_WAVES * 64) {  // (more than once with more than 8 heads)
        const int item = min(i0 + (parts > 1 ? tid % items : tid), items - 1), part = parts > 1 ? tid / items : 0;
        const float* pp = address(item);
        uint2 x[DENSE_BATCH];
        if (part < parts) {
#pragma unroll
            for (int k = 0; k < DENSE_BATCH; ++k) {
                const int s = part + k * parts;
                x[k] = s < ns ? ld_dev_u2(pp + (int64_t)s * HATA_PSTRIDE) : make_uint2(0, 0);
            }
        }
        if (i0 == 0) {
            for (int g = wave; g < G; g += DENSE_WAVES) {
                const float* mp = part0 + g * head_stride;
                uint2 ml[4];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (t * 64 < ns) ml[t] = ld_dev_u2(mp + (int64_t)min(lane + 64 * t, ns - 1) * HATA_PSTRIDE);
                float M = HATA_NEG_INF;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (lane + 64 * t < ns) M = fmaxf(M, __uint_as_float(ml[t].x));
                M = wave_max64(M);
                float w[4], l = 0.f;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    w[t] = lane + 64 * t < ns && M != HATA_NEG_INF ? fast_exp2(__uint_as_float(ml[t].x) - M) : 0.f;
                    if (lane + 64 * t < ns) l = fmaf(w[t], __uint_as_float(ml[t].y), l);
                }
                l = wave_sum64(l);
                const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (lane + 64 * t < ns) s_w[g * ns + lane + 64 * t] = w[t] * inv;
            }
            __syncthreads();
        }
        float2 sum = make_float2(0.f, 0.f);
        if (part < parts) {
            const float* w = s_w + item / (HATA_D / 2) * ns;
            for (int s0 = part;;) {
#pragma unroll
                for (int k = 0; k < DENSE_BATCH; ++k) {
                    const float f = w[min(s0 + k * parts, ns - 1)];  // (x is zero past the end)
                    sum.x = fmaf(f, __uint_as_float(x[k].x), sum.x);
                    sum.y = fmaf(f, __uint_as_float(x[k].y), sum.y);
                }
                s0 += DENSE_BATCH * parts;
                if (s0 >= ns) break;
#pragma unroll
                for (int k = 0; k < DENSE_BATCH; ++k) {
                    const int s = s0 + k * parts;
                    x[k] = s < ns ? ld_dev_u2(pp + (int64_t)s * HATA_PSTRIDE) : make_uint2(0, 0);
                }
            }
        }
        if (parts > 1) {  // (a single turn)
            if (part < parts) s_sum[part * items + item] = sum;
            __syncthreads();
            if (part > 0) return;
            for (int k = 1; k < parts; ++k) {
                sum.x += s_sum[k * items + item].x;
                sum.y += s_sum[k * items + item].y;
            }
        } else if (i0 + tid >= items) {
            return;
        }
        outp[2 * item] = (uint16_t)f32_to_bf16(sum.x);
        outp[2 * item + 1] = (uint16_t)f32_to_bf16(sum.y);
        if (outp32) { outp32[2 * item] = sum.x; outp32[2 * item + 1] = sum.y; }
    }
}

static size_t dense_lds() { return (size_t)DENSE_WAVES * DENSE_RING * DENSE_TILE_BYTES; }

// Workgroups per unit: the launch runs in rounds of one workgroup per CU, each as long as its rows and a fixed
// cost worth about as much as 256 rows (launch, first request, merge); at most HATA_DENSE_ROUNDS rounds.
static int dense_splits(int64_t units, int L_cap) {
    int best = 1;
    int64_t best_cost = INT64_MAX;
    for (int m = 0; m <= HATA_DENSE_ROUNDS; ++m) {
        const int64_t s = m == 0 ? 1 : std::min(256 * m / units, (int64_t)std::min(DENSE_MAX_RUNS, (L_cap + 127) / 128));
        if (s < 1) continue;
        const int64_t cost = (units * s + 256 - 1) / 256 * ((L_cap + s - 1) / s + 256);
        if (cost < best_cost) { best_cost = cost; best = (int)s; }
    }
    return best;
}

hipError_t prepare_dense() {  // (more than 64 KB of dynamic LDS has to be asked for)
    for (const void* fn : {(const void*)dense_kernel<DENSE_BF16X2>, (const void*)dense_kernel<DENSE_FP32>,
                           (const void*)dense_kernel<DENSE_FP32_ONE_HEAD>, (const void*)dense_kernel<DENSE_FP32_TWO_HEADS>}) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dense_lds());
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_dense(const hata_ctx* c, const void* q, const void* K, const void* V, const int32_t* seq_len, int B,
                        float sm_scale, void* out, float* out_f32, hipStream_t s) {
    const hata_config& f = c->cfg;
    DenseArgs a;
    a.q = (const uint16_t*)q; a.K = (const uint16_t*)K; a.V = (const uint16_t*)V;
    a.seq_len = seq_len;
    a.partials = c->partials; a.counter = c->attn_counter; a.counter_stride = c->attn_counter_stride;
    a.out = (uint16_t*)out; a.out_f32 = out_f32;
    a.Hq = f.Hq; a.Hkv = f.Hkv; a.G = c->G; a.L_cap = f.L_cap;
    a.B = B;
    // one run a unit is even only among sequences of one length: workgroups to spare for the long ones
    const int64_t units = (int64_t)f.Hkv * B, splits = dense_splits(units, f.L_cap);
    const int64_t spare = splits == 1 && B > 1 ? std::max((int64_t)0, std::min((int64_t)256, c->dense_wgs_max - units)) : 0;
    a.sb = f.kv_stride_b; a.sh = f.kv_stride_h; a.sn = f.kv_stride_n;
    a.scale_log2 = sm_scale * 1.4426950408889634f;
    const dim3 grid = B == 1 ? dim3((unsigned)splits, f.Hkv) : dim3((unsigned)(units * splits + spare));
    const auto fn = c->HT >= 4 ? dense_kernel<DENSE_BF16X2> : c->G == 1 ? dense_kernel<DENSE_FP32_ONE_HEAD>
                    : c->G == 2 ? dense_kernel<DENSE_FP32_TWO_HEADS> : dense_kernel<DENSE_FP32>;
    hipLaunchKernelGGL(fn, grid, dim3(DENSE_WAVES * 64), dense_lds(), s, a);
    return hipGetLastError();
}

}  // namespace hata
