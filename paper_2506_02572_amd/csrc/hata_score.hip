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
// (hata_attn.hip).  encode_score_kernel is the same with the encoding in it, where one round of large workgroups covers the batch; with
// workgroups of 256 threads, a chunk each, it was 3.9 us of the kernel, more than the launch in front takes.
#include <type_traits>

#include "hata_device.h"
#include "hata_hash.h"
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
// next launch looks for the threshold.  256 threads (t), after a barrier; scan4: 4 words of LDS.  Whoever is not `live` passes the
// barrier only.
__device__ __forceinline__ void store_cumulative(const ScoreArgs& a, const uint32_t* hist, int64_t u, int c, int b, int L, uint32_t* scan4,
                                                 int t, bool live = true) {
    uint16_t* const row = a.cum + (u * a.n_chunks + c) * a.NBP;
    const int NBP = a.NBP, NBR = (a.NB + 15) / 16 * 16, n_keys = min(a.chunk, L - c * a.chunk);
    const int keff = min(clampi(a.kbud[b], 0, a.k_max), L);
    const uint32_t share = (uint32_t)min(n_keys, (int)((float)keff * (float)n_keys * __builtin_amdgcn_rcpf((float)L)) + 1);
    const int wv = t >> 6, seg = ((NBR + 255) / 256 + 3) / 4 * 4, s0 = t * seg;
    uint32_t loc = 0;
    for (int j = 0; live && j < seg; j += 4)
        if (s0 + j < NBR) {
            const uint4 v = *reinterpret_cast<const uint4*>(&hist[s0 + j]);
            loc += v.x + v.y + v.z + v.w;
        }
    const uint32_t incl = wave_incl_scan(loc);
    if (live && (t & 63) == 63) scan4[wv] = incl;
    __syncthreads();
    if (!live) return;
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
    store_cumulative(a, hist, u, c, b, L, scan4, tid);
}

struct EncodeScoreArgs {
    ScoreArgs s;
    const uint16_t* q;
    const uint16_t* K;
    const float* W_H;
    uint32_t* codes;
    uint32_t* qcodes;
    int append, log2_chunks;  // of a workgroup, by the cache's size
    int64_t sb, sh, sn;
};

// Where the cache's size gives a workgroup four chunks: how few the sequences' lengths allow in the same grid, and which workgroup of which
// sequence this one is then; each sequence has one at least, which writes its query codes.  By position alone a long sequence among short ones was
// left to a quarter of the workgroups while most compute units had nothing (r = 128, 16 sequences, one of 32768 keys, the others of 500,
// us a step: two launches 41.4, by position 43.6, so 38.4; groups of eight 47.6, 50.4, 44.6; all of 16384, 47.3, 45.0, 40.5; all full 46.5, 44.7,
// 45.5).  Where no less than four will do the places are those by position.  own: sequence lane's length, loaded ahead of the weights;
// false: nothing left for this one.
struct EncodeScorePlace { int b, x, log2_chunks, length; };
__device__ __forceinline__ bool place_by_length(const ScoreArgs& a, int own, EncodeScorePlace& at) {
    const int lane = threadIdx.x & 63, B = gridDim.z, slots = gridDim.x * B, log2_chunk = __builtin_ctz(a.chunk);
    auto length_of = [&](int b0) { return b0 == 0 ? own : a.seq_len[min(b0 + lane, B - 1)]; };
    auto workgroups = [&](int b0) {
        const int n = (clampi(length_of(b0), 0, a.L_cap) + a.chunk - 1) >> log2_chunk;
        return b0 + lane < B ? (uint32_t)max((n + (1 << at.log2_chunks) - 1) >> at.log2_chunks, 1) : 0u;
    };
    uint32_t upto;  // workgroups of the sequences up to this lane's, of the last 64 looked at
    for (at.log2_chunks = 0; at.log2_chunks < 2; ++at.log2_chunks) {
        int n = 0;
        for (int b0 = 0; b0 < B; b0 += 64) {
            upto = wave_incl_scan(workgroups(b0));
            n += __builtin_amdgcn_readlane((int)upto, 63);
        }
        if (n <= slots) break;
    }
    if (at.log2_chunks == 2) {  // by position
        at.b = blockIdx.z;
        at.x = blockIdx.x;
        at.length = __builtin_amdgcn_readlane(length_of(at.b & ~63), at.b & 63);
        return true;
    }
    int left = blockIdx.z * gridDim.x + blockIdx.x;
    for (int b0 = 0; b0 < B; b0 += 64) {
        if (B > 64) upto = wave_incl_scan(workgroups(b0));
        const int n = __builtin_amdgcn_readlane((int)upto, 63);
        if (left < n) {
            const int l = __builtin_ctzll(__builtin_amdgcn_ballot_w64((int)upto > left));
            at.b = b0 + l;
            at.x = left - (l ? __builtin_amdgcn_readlane((int)upto, max(l - 1, 0)) : 0);
            at.length = __builtin_amdgcn_readlane(length_of(b0), l);
            return true;
        }
        left -= n;
    }
    return false;
}

// The scoring launch with the encoding in it: a workgroup of 1024 threads encodes its unit's query vectors for itself (and the appended
// key, where its chunks hold that row) as the workgroup per unit of hata_unit.hip does, its first codes on their way meanwhile, and
// then has 1024, 512 or 256 threads for each of one, two or four chunks.  grid = (workgroups of a unit, Hkv, B); FOUR: dealt out by the lengths
// (which costs two chunks a workgroup 0.4 us a launch and saves them less).
// What bounds it: the launch, the round trips to the weights and the appended row, half a microsecond of fp64 of every compute unit.
// A launch in front of the scoring costs its own launch and round trips on top: 2 x 20011 keys, a group of five, 21.7 us a step with one,
// 20.2 so (launch_encode_score has the rule).
template <int WD, int G, bool FOUR>
__global__ __launch_bounds__(1024) void encode_score_kernel(const EncodeScoreArgs a) {
    constexpr int R = WD * 32, NB = G * R + 1, NBR = (NB + 15) / 16 * 16, NW = 16, NT = 1024;
    constexpr int PASSES = G / 4 + 1;  // of four vectors: the query heads and the appended key, which goes alone where the heads fill theirs
    constexpr int UNR = 4;             // keys of a thread whose codes are in flight together
    using Hash = UnitHash<R>;
    static_assert(Hash::PARTS > 1, "the waves of a group of columns meet in LDS");
    __shared__ double part[PASSES][NW][64];
    __shared__ uint32_t s_codes[(G + 1) * WD];
    __shared__ uint32_t scan4[4][4];
    extern __shared__ __attribute__((aligned(16))) uint32_t hists[];  // [chunks of the workgroup][NBR]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.y;
    EncodeScorePlace at;
    int own_length = 0;
    if constexpr (FOUR) own_length = a.s.seq_len[min(lane, (int)gridDim.z - 1)];
    Hash hash;
    hash.fetch(a.W_H + (int64_t)h * HATA_D * R);
    if constexpr (FOUR) {
        if (!place_by_length(a.s, own_length, at)) return;
    } else {
        at = {(int)blockIdx.z, (int)blockIdx.x, a.log2_chunks, 0};
    }
    const int b = at.b, log2_threads = 10 - at.log2_chunks;
    const int64_t u = (int64_t)b * a.s.Hkv + h;
    const uint16_t* qv = a.q + ((int64_t)b * a.s.Hq + (int64_t)h * G) * HATA_D;
    typename Hash::Vector x[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p)
        if (4 * p < G) x[p] = Hash::fetch_x(qv + min(4 * p + (lane & 3), G - 1) * HATA_D);
    if constexpr (!FOUR) at.length = a.s.seq_len[b];
    const int L = clampi(at.length, 0, a.s.L_cap);
    const int chunks = NT >> log2_threads, threads = 1 << log2_threads, sub = tid >> log2_threads, t = tid & (threads - 1);
    const int first = at.x * chunks * a.s.chunk;
    if (first >= L && at.x != 0) return;  // (the first workgroup writes the query codes of an empty sequence too)
    const int c = at.x * chunks + sub, base = c * a.s.chunk, end = min(base + a.s.chunk, L);
    // row L - 1 is encoded here (a sequence longer than its cache appends a row that is not there)
    const bool own = a.append && at.length <= a.s.L_cap && L - 1 >= first && L - 1 < first + chunks * a.s.chunk;
    if (own) {
        const uint16_t* kx = a.K + b * a.sb + h * a.sh + (int64_t)(L - 1) * a.sn;
        if (G % 4 == 0 || (lane & 3) == G % 4) x[PASSES - 1] = Hash::fetch_x(kx);
    }
    const uint32_t* const cp = a.s.codes + u * a.s.L_cap * WD;
    const int stop = own ? min(end, L - 1) : end;
    CodeVec<WD> kc[UNR];
    auto load_codes = [&](int n0) {
#pragma unroll
        for (int j = 0; j < UNR; ++j) {
            const int n = n0 + j * threads;
            if (n < stop) kc[j] = load_code<WD>(cp + (int64_t)n * WD);
        }
    };
    load_codes(base + t);
    for (int i = tid; i < chunks * NBR; i += NT) hists[i] = 0;
    const int vectors = own ? G + 1 : G, group = wave % Hash::GROUPS;
    auto there = [&](int p) { return 4 * p < G || own; };
#pragma unroll
    for (int p = 0; p < PASSES; ++p)
        if (there(p)) part[p][wave][lane] = 4 * p < G ? hash.project(x[p]) : hash.project_one(x[p]);
    __syncthreads();
    // the waves of a group of columns share the passes
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        if (there(p) && p % Hash::PARTS == wave / Hash::GROUPS) {
            double v = part[p][group][lane];
#pragma unroll
            for (int i = 1; i < Hash::PARTS; ++i) v += part[p][group + i * Hash::GROUPS][lane];
            if (4 * p < G) Hash::store_bits(v, s_codes, group, 4 * p, vectors);
            else Hash::store_bits_one(v, s_codes, group, G);
        }
    }
    __syncthreads();
    if (at.x == 0 && tid < G * WD) a.qcodes[((int64_t)b * a.s.Hq + (int64_t)h * G) * WD + tid] = s_codes[tid];
    if (own && tid < WD) a.codes[(u * a.s.L_cap + L - 1) * WD + tid] = s_codes[G * WD + tid];
    QuerySum<WD, G> sum;
    sum.init(s_codes);
    uint32_t* const hist = hists + sub * NBR;
    uint16_t* const sp = a.s.scores + u * a.s.L_cap;
    auto scored = [&](int n, const uint32_t (&k)[WD]) {
        const uint32_t s = sum(k);
        sp[n] = (uint16_t)s;
        atomicAdd(&hist[s], 1u);
    };
    for (int n0 = base + t; n0 < stop;) {
#pragma unroll
        for (int j = 0; j < UNR; ++j)
            if (n0 + j * threads < stop) scored(n0 + j * threads, kc[j].w);
        n0 += threads * UNR;
        if (n0 < stop) load_codes(n0);
    }
    if (own && t == 0 && L - 1 >= base && L - 1 < base + a.s.chunk) {
        uint32_t kw[WD];
#pragma unroll
        for (int w = 0; w < WD; ++w) kw[w] = s_codes[G * WD + w];
        scored(L - 1, kw);
    }
    __syncthreads();
    store_cumulative(a.s, hist, u, c, b, L, scan4[sub], t, base < L && t < 256);
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
        store_cumulative(a, hist, u, c, b, L, scan4, tid);
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

template <int WD, bool FOUR>
static const void* encode_score_fn(int G) {
    switch (G) {
        case 1: return (const void*)&encode_score_kernel<WD, 1, FOUR>;
        case 2: return (const void*)&encode_score_kernel<WD, 2, FOUR>;
        case 4: return (const void*)&encode_score_kernel<WD, 4, FOUR>;
        case 5: return (const void*)&encode_score_kernel<WD, 5, FOUR>;
        case 8: return (const void*)&encode_score_kernel<WD, 8, FOUR>;
        default: return nullptr;
    }
}

// query codes, the appended key's code, scores and cumulative chunk histograms in one launch; hipErrorNotSupported: not this shape
hipError_t launch_encode_score(const hata_ctx* c, const void* q, const void* K, const float* W_H, uint32_t* codes, int append,
                               const int32_t* seq_len, const int32_t* k, int B, hipStream_t s) {
    const hata_config& f = c->cfg;
    // One round of workgroups, with as few chunks each as that allows: in more, every one of them encodes on the bandwidth's time (us a
    // step, two launches / one: 160 units of 4096-key chunks, 32768 keys 49.6 / 52.1, 40 units of 131072 45.2 / 51.5; one head a
    // unit, 256 of 32768, 64.9 / 64.0).  Up to it, r = 128: 8 units of 32768 keys 20.1 / 17.8, of 131072 23.9 / 21.1, 32 of
    // 16000 21.3 / 19.1, groups of eight 16 of 32768 25.5 / 23.3, four chunks a workgroup 128 of 32768 45.4 / 42.9, one head a unit 33.1 / 31.9.
    // r = 64 and 32, 8 units of 32768 keys: groups of four 19.1 / 16.6 and 19.0 / 16.1, of eight 25.6 / 22.7 and 25.4 / 21.8, one head 15.9 / 14.5 and
    // 15.7 / 13.9; four chunks a workgroup, one head, 32 units of 131072 30.7 / 29.5 and 28.2 / 26.5 (r = 128 38.8 / 39.1).
    // r = 256 has twice the fp64, and the weights leave no registers to hide it behind the codes' loads: 8 units of 20000 keys 19.8 / 19.8, two
    // heads a unit 19.2 / 20.0, 32 units of 131072 45.0 / 45.5, groups of eight 24.4 / 27.0 -- it keeps two launches.
    int chunks = 1;
    auto wgs = [&](int n) { return (int64_t)((c->n_chunks + n - 1) / n) * f.Hkv * B; };
    while (chunks < 4 && wgs(chunks) > c->cus) chunks *= 2;
    auto of_width = [&](auto four) {
        constexpr bool F = decltype(four)::value;
        return c->Wd == 1 ? encode_score_fn<1, F>(c->G) : c->Wd == 2 ? encode_score_fn<2, F>(c->G) : c->Wd == 4 ? encode_score_fn<4, F>(c->G) : nullptr;
    };
    const void* fn = chunks == 4 ? of_width(std::true_type{}) : of_width(std::false_type{});
    if (!fn || wgs(chunks) > c->cus) return hipErrorNotSupported;
    EncodeScoreArgs a;
    a.s = score_args(c, c->qcodes, codes, seq_len, c->scores, k);
    a.q = (const uint16_t*)q; a.K = (const uint16_t*)K; a.W_H = W_H; a.codes = codes; a.qcodes = c->qcodes;
    a.append = append;
    a.log2_chunks = __builtin_ctz(chunks);
    a.sb = f.kv_stride_b; a.sh = f.kv_stride_h; a.sn = f.kv_stride_n;
    void* args[] = {(void*)&a};
    return hipLaunchKernel(fn, dim3((c->n_chunks + chunks - 1) / chunks, f.Hkv, B), dim3(1024), args, (size_t)chunks * ((c->NB + 15) / 16 * 64), s);
}

}  // namespace hata
