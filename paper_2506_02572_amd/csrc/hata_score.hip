// Hamming-score kernel (Alg. 3 of the paper: S = bitcount(xor(Q_H, K_H^cache)), summed
// over the query heads of a GQA group so that the group shares ONE pass over the codes).
//
// Bandwidth-bound streaming: each lane owns one cached key per iteration and pulls its
// whole packed code with 128-bit loads (a wave reads 1 KB or 2 KB of consecutive bytes);
// the G query codes are wave-uniform and sit in scalar registers.
//
// score_select_kernel is the scoring launch of the decode step without in-kernel waits: the workgroup also histograms its
// chunk's scores in LDS and writes the CUMULATIVE histogram out (how many of the chunk's keys score at most s, 2 bytes per
// s), from which the workgroups of the attention launch find the unit's threshold and their places in the index list
// (hata_attn.hip).  (Every workgroup encoding its unit's queries for itself instead of a launch in front: 3.9 us of the
// kernel, more than the launch takes: 2 x 20011 keys, a group of five, 23.7 us a step against 22.2.)
#include "hata_device.h"
#include "hata_internal.h"
#include "hata_trace.h"

namespace hata {

template <int WD>
struct CodeVec { uint32_t w[WD]; };

template <int WD>
__device__ __forceinline__ CodeVec<WD> load_code(const uint32_t* p) {
    CodeVec<WD> c;
    if constexpr (WD % 4 == 0) {
#pragma unroll
        for (int i = 0; i < WD / 4; ++i) {
            uint4 v = reinterpret_cast<const uint4*>(p)[i];
            c.w[4 * i] = v.x; c.w[4 * i + 1] = v.y; c.w[4 * i + 2] = v.z; c.w[4 * i + 3] = v.w;
        }
    } else if constexpr (WD % 2 == 0) {
#pragma unroll
        for (int i = 0; i < WD / 2; ++i) {
            uint2 v = reinterpret_cast<const uint2*>(p)[i];
            c.w[2 * i] = v.x; c.w[2 * i + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < WD; ++i) c.w[i] = p[i];
    }
    return c;
}

// scores of rows n0, n0 + 256, ... < end of a unit (cp: its codes), handed to each(n, score)
template <int WD, int G, typename Sum, typename Each>
__device__ __forceinline__ void score_rows(const uint32_t* cp, int n0, int end, const Sum& sum, Each each) {
    constexpr int UNR = (WD <= 4) ? 8 : 4;  // 128 B of codes in flight per lane (256 B measured: 0.3-1 us slower)
    for (; n0 < end; n0 += 256 * UNR) {
        CodeVec<WD> kc[UNR];
#pragma unroll
        for (int j = 0; j < UNR; ++j) {
            const int n = n0 + j * 256;
            if (n < end) kc[j] = load_code<WD>(cp + (int64_t)n * WD);
        }
#pragma unroll
        for (int j = 0; j < UNR; ++j) {
            const int n = n0 + j * 256;
            if (n < end) each(n, sum(kc[j].w));
        }
    }
}

// wave-uniform query codes: as they are, or as bit-count planes for the larger groups
template <int WD, int G>
struct QuerySum {
    static constexpr bool PLANES = HammingSum<WD, G>::PLANES;
    HammingSum<WD, G> dist;
    uint32_t qc[PLANES ? 1 : G][WD];
    __device__ __forceinline__ void init(const uint32_t* qp) {
        if constexpr (PLANES) {
            dist.init(qp);
        } else {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int w = 0; w < WD; ++w) qc[g][w] = __builtin_amdgcn_readfirstlane(qp[g * WD + w]);
        }
    }
    __device__ __forceinline__ uint32_t operator()(const uint32_t (&k)[WD]) const {
        if constexpr (PLANES) {
            return dist(k);
        } else {
            uint32_t s = 0;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int w = 0; w < WD; ++w) s += __popc(qc[g][w] ^ k[w]);
            return s;
        }
    }
};

template <int WD, int G>
__global__ __launch_bounds__(256) void score_kernel(
    const uint32_t* __restrict__ qcodes, const uint32_t* __restrict__ codes, const int32_t* __restrict__ seq_len,
    uint16_t* __restrict__ scores, int Hq, int Hkv, int L_cap, int chunk) {
    const int tid = threadIdx.x, c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    // (the query codes' loads do not depend on the sequence length and go out together with it)
    QuerySum<WD, G> sum;
    sum.init(qcodes + ((int64_t)b * Hq + (int64_t)h * G) * WD);
    const int L = clampi(seq_len[b], 0, L_cap);
    const int base = c * chunk, end = min(base + chunk, L);
    const int64_t u = (int64_t)b * Hkv + h;
    uint16_t* sp = scores + u * L_cap;
    score_rows<WD, G>(codes + u * L_cap * WD, base + tid, end, sum, [&](int n, uint32_t s) { sp[n] = (uint16_t)s; });
}

struct ScoreArgs {
    const uint32_t* qcodes;
    const uint32_t* codes;
    const int32_t* seq_len;
    uint16_t* scores;
    uint16_t* cum;         // [units, n_chunks, NBP]
    int32_t* estimate;     // [units, n_chunks]
    const int32_t* kbud;   // nullptr: scores only
    int Hq, Hkv, L_cap, chunk, n_chunks, NB, NBP, k_max;
};

// The chunk's histogram in LDS (a multiple of 16 words, zero past its NB scores) -> its row of cumulative counts, and
// the score at which these reach the chunk's share of the budget, if that were spread evenly over the unit's L keys: where the
// next launch looks for the threshold.  256 threads, after a barrier; scan4: 4 words of LDS.
__device__ __forceinline__ void store_cumulative(const ScoreArgs& a, const uint32_t* hist, int64_t u, int c, int b, int L, uint32_t* scan4) {
    uint16_t* const row = a.cum + (u * a.n_chunks + c) * a.NBP;
    const int NBP = a.NBP, NBR = (a.NB + 15) / 16 * 16, n_keys = min(a.chunk, L - c * a.chunk);
    const int keff = min(clampi(a.kbud[b], 0, a.k_max), L);
    const uint32_t share = (uint32_t)min(n_keys, (int)((float)keff * (float)n_keys * __builtin_amdgcn_rcpf((float)L)) + 1);
    const int tid = threadIdx.x, wv = tid >> 6, seg = ((NBR + 255) / 256 + 3) / 4 * 4, s0 = tid * seg;
    uint32_t loc = 0;
    for (int j = 0; j < seg; j += 4)
        if (s0 + j < NBR) {
            const uint4 v = *reinterpret_cast<const uint4*>(&hist[s0 + j]);
            loc += v.x + v.y + v.z + v.w;
        }
    const uint32_t incl = wave_incl_scan(loc);
    if ((tid & 63) == 63) scan4[wv] = incl;
    __syncthreads();
    uint32_t run = (wv > 0 ? scan4[0] : 0u) + (wv > 1 ? scan4[1] : 0u) + (wv > 2 ? scan4[2] : 0u) + incl - loc;
    for (int j = 0; j < seg; j += 4)
        if (s0 + j < NBP) {
            const uint4 v = s0 + j < NBR ? *reinterpret_cast<const uint4*>(&hist[s0 + j]) : make_uint4(0, 0, 0, 0);
            const uint32_t c0 = run + v.x, c1 = c0 + v.y, c2 = c1 + v.z, c3 = c2 + v.w;
            if (run < share && c3 >= share)
                a.estimate[u * a.n_chunks + c] = s0 + j + (c0 < share ? 1 : 0) + (c1 < share ? 1 : 0) + (c2 < share ? 1 : 0);
            run = c3;
            *reinterpret_cast<uint2*>(row + s0 + j) = make_uint2(c0 | (c1 << 16), c2 | (c3 << 16));
        }
}

// grid = (n_chunks, Hkv, B)
template <int WD, int G>
__global__ __launch_bounds__(256) void score_select_kernel(const ScoreArgs a) {
    constexpr int NB = G * WD * 32 + 1, NBR = (NB + 15) / 16 * 16;
    __shared__ __attribute__((aligned(16))) uint32_t hist[NBR];
    __shared__ uint32_t scan4[4];
    const int tid = threadIdx.x, c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int64_t u = (int64_t)b * a.Hkv + h;
    const int base = c * a.chunk;
    QuerySum<WD, G> sum;
    sum.init(a.qcodes + ((int64_t)b * a.Hq + (int64_t)h * G) * WD);
    const int L = clampi(a.seq_len[b], 0, a.L_cap);
    if (base >= L) return;
    for (int i = tid; i < NBR; i += 256) hist[i] = 0;
    __syncthreads();
    const int end = min(base + a.chunk, L);
    uint16_t* sp = a.scores + u * a.L_cap;
    score_rows<WD, G>(a.codes + u * a.L_cap * WD, base + tid, end, sum, [&](int n, uint32_t s) {
        sp[n] = (uint16_t)s;
        atomicAdd(&hist[s], 1u);
    });
    __syncthreads();
    store_cumulative(a, hist, u, c, b, L, scan4);
}

// Generic fallback: any WD <= 8 and G <= 16, query codes in LDS.
__global__ __launch_bounds__(256) void score_kernel_generic(const ScoreArgs a, int G, int WD) {
    extern __shared__ __attribute__((aligned(16))) uint32_t hist[];
    __shared__ uint32_t qc[16 * 8];
    __shared__ uint32_t scan4[4];
    const int tid = threadIdx.x, c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int L = clampi(a.seq_len[b], 0, a.L_cap);
    const int base = c * a.chunk, NBR = (a.NB + 15) / 16 * 16;
    const int64_t u = (int64_t)b * a.Hkv + h;
    if (base >= L) return;
    const int end = min(base + a.chunk, L);
    for (int i = tid; i < NBR; i += 256) hist[i] = 0;
    if (tid < G * WD) qc[tid] = a.qcodes[((int64_t)b * a.Hq + (int64_t)h * G) * WD + tid];
    __syncthreads();
    const uint32_t* cp = a.codes + u * a.L_cap * WD;
    uint16_t* sp = a.scores + u * a.L_cap;
    for (int n = base + tid; n < end; n += 256) {
        uint32_t s = 0;
        for (int w = 0; w < WD; ++w) {
            const uint32_t kw = cp[(int64_t)n * WD + w];
            for (int g = 0; g < G; ++g) s += __popc(qc[g * WD + w] ^ kw);
        }
        sp[n] = (uint16_t)s;
        if (a.kbud) atomicAdd(&hist[s], 1u);
    }
    if (a.kbud) {
        __syncthreads();
        store_cumulative(a, hist, u, c, b, L, scan4);
    }
}

static ScoreArgs score_args(const hata_ctx* c, const uint32_t* qcodes, const uint32_t* codes, const int32_t* seq_len, uint16_t* scores,
                            const int32_t* kbud) {
    const hata_config& f = c->cfg;
    ScoreArgs a = {};
    a.qcodes = qcodes; a.codes = codes; a.seq_len = seq_len; a.scores = scores;
    a.cum = c->chunk_hist; a.estimate = c->chunk_info; a.kbud = kbud; a.k_max = f.k_max;
    a.Hq = f.Hq; a.Hkv = f.Hkv; a.L_cap = f.L_cap; a.chunk = c->chunk; a.n_chunks = c->n_chunks; a.NB = c->NB; a.NBP = c->NBP;
    return a;
}
static void launch_generic(const hata_ctx* c, const ScoreArgs& a, int B, hipStream_t s) {
    hipLaunchKernelGGL(score_kernel_generic, dim3(c->n_chunks, c->cfg.Hkv, B), dim3(256), (size_t)(c->NB + 15) / 16 * 64, s, a, c->G, c->Wd);
}

#define HATA_SCORE_CASES                                                                                      \
    HATA_CASE(4, 1) HATA_CASE(4, 2) HATA_CASE(4, 4) HATA_CASE(4, 5) HATA_CASE(4, 8)                           \
    HATA_CASE(8, 1) HATA_CASE(8, 2) HATA_CASE(8, 4) HATA_CASE(8, 5) HATA_CASE(8, 8)                           \
    HATA_CASE(2, 1) HATA_CASE(2, 2) HATA_CASE(2, 4) HATA_CASE(2, 5) HATA_CASE(2, 8)                           \
    HATA_CASE(1, 1) HATA_CASE(1, 2) HATA_CASE(1, 4) HATA_CASE(1, 5) HATA_CASE(1, 8)                           \
    HATA_CASE(1, 16) HATA_CASE(2, 16) HATA_CASE(4, 16) HATA_CASE(8, 16)

// scores only
hipError_t launch_score(const hata_ctx* c, const uint32_t* qcodes, const uint32_t* codes, const int32_t* seq_len, int B,
                        uint16_t* scores, hipStream_t s) {
    const hata_config& f = c->cfg;
    const dim3 grid(c->n_chunks, f.Hkv, B);
    switch (c->Wd * 100 + c->G) {
#define HATA_CASE(WD, GG)                                                                                     \
    case WD * 100 + GG:                                                                                       \
        hipLaunchKernelGGL((score_kernel<WD, GG>), grid, dim3(256), 0, s, qcodes, codes, seq_len, scores,     \
                           f.Hq, f.Hkv, f.L_cap, c->chunk);                                                   \
        break;
        HATA_SCORE_CASES
#undef HATA_CASE
        default: launch_generic(c, score_args(c, qcodes, codes, seq_len, scores, nullptr), B, s);
    }
    return hipGetLastError();
}

// scores and cumulative chunk histograms into the workspace
hipError_t launch_score_select(const hata_ctx* c, const uint32_t* codes, const int32_t* seq_len, const int32_t* k, int B, hipStream_t s) {
    const ScoreArgs a = score_args(c, c->qcodes, codes, seq_len, c->scores, k);
    const dim3 grid(c->n_chunks, c->cfg.Hkv, B);
    switch (c->Wd * 100 + c->G) {
#define HATA_CASE(WD, GG) \
    case WD * 100 + GG: hipLaunchKernelGGL((score_select_kernel<WD, GG>), grid, dim3(256), 0, s, a); break;
        HATA_SCORE_CASES
#undef HATA_CASE
        default: launch_generic(c, a, B, s);
    }
    return hipGetLastError();
}

}  // namespace hata
