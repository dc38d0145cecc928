// Decode step over a short cache: a workgroup of 1024 threads does everything for one (sequence, KV head) unit -- hash
// encoding, Hamming scores, top-k selection and attention over the selected rows (Alg. 3 of the paper).
//
// What bounds the step over a few thousand keys is neither bytes nor operations but the chain of exchanges between the
// workgroups that share a unit (hata_coop.hip).  With up to 4096 keys a compute unit reads a unit's codes (64 KB at
// r = 128) in the time of one or two exchanges, so nothing is shared: every stage hands over in LDS, a barrier
// apart.  No workgroup waits for another one either, so the grid need not be resident and the device may be shared.
// us a layer, workgroups that share units / this: one sequence, eight KV heads, r = 128, 2048 keys 16.0 / 10.3, 4096 keys
// 15.7 / 11.3, a group of eight 19.6 / 13.7, r = 256 18.2 / 14.8; 32 sequences of 4096 keys 22.8 / 13.5.
// Beyond that the unit's time is what one compute unit streams and gathers, so longer caches and large budgets take this
// form only where the units are many: takes_unit_step in hata_api.hip, with both sides measured.
#include "hata_attn_core.h"
#include "hata_device.h"
#include "hata_hash.h"
#include "hata_internal.h"

namespace hata {

#define HATA_UNIT_WAVES 16
#define HATA_UNIT_THREADS (HATA_UNIT_WAVES * 64)

struct UnitArgs {
    const uint16_t* q;
    const uint16_t* K;
    const uint16_t* V;
    const float* W_H;
    const int32_t* seq_len;
    const int32_t* kbud;
    uint32_t* codes;
    uint32_t* qcodes;
    uint16_t* scores;  // nullptr: not wanted
    int32_t* idx;
    uint16_t* out;
    float* out_f32;
    int Hq, Hkv, L_cap, k_max, append;
    int log2_kpt;  // consecutive keys of a thread (LONG)
    int64_t sb, sh, sn;
    float scale_log2;
    PageView pv;  // block table (used by the PAGED instantiations only)
};

// sum over the waves before this one of a value per wave (tot: 16 words of LDS, complete), and over all of them
__device__ __forceinline__ uint32_t before_wave(const uint32_t* tot, uint32_t& all) {
    const uint32_t incl = wave_incl_scan(tot[threadIdx.x & 15]);  // (lanes 0..15 of every wave)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 15);
    return wave == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)incl, wave - 1);
}

// LONG: more than HATA_UNIT_KEYS keys, a power of two kpt = 8 or 16 of consecutive ones per thread.  A thread's scores lie in
// LDS a word (two of them) from every row of 1024 words, turned by four words a row, so that neither the writes -- 64 consecutive
// keys of a wave -- nor a thread's reads of its own keys meet in a bank.
template <int WD, int G, bool PAGED, bool LONG>
__global__ __launch_bounds__(HATA_UNIT_THREADS) void decode_step_unit_kernel(const UnitArgs a) {
    constexpr int R = WD * 32, NB = G * R + 1, NBR = (NB + 15) / 16 * 16;
    constexpr int NW = HATA_UNIT_WAVES, NT = HATA_UNIT_THREADS;
    constexpr int MAX_KEYS = LONG ? HATA_UNIT_KEYS_LONG : HATA_UNIT_KEYS;
    constexpr int UNR = LONG && WD <= 4 ? 8 : 4;  // keys of a thread whose codes are in flight together
    constexpr bool MFMA = G >= 4;             // matrix-core form of the attention core
    using Hash = UnitHash<R>;
    // Passes of four vectors, the query heads and the appended key.  Where the heads fill theirs, the key's goes over the vector
    // ALU: alone it took the matrix instruction as long as four (16.6 cycles for an fp64 FMA's 4.4), and the waves of a compute unit were
    // 0.45 us at it (us a layer, groups of four: 2048 keys 10.98 -> 10.57, 4096 11.88 -> 11.52, r = 256 14.61 -> 14.05; of eight
    // 13.54 -> 13.08, 128 units of 4096 keys 16.01 -> 15.66).  One or two left-over heads too: no faster (11.85 / 12.05, a group of five).
    constexpr int PASSES = G / 4 + 1;
    __shared__ __attribute__((aligned(16))) union {
        double part[PASSES][NW][64];  // projections, by the waves that share their columns
        uint16_t vt[MFMA ? NW * HATA_VT_WAVE : 8];
        AttnLds<G, LONG ? NW : 1> s;
    } U;
    __shared__ __attribute__((aligned(16))) AttnLds<G, LONG ? 1 : NW> S_own;
    AttnLds<G, NW>& S = *reinterpret_cast<AttnLds<G, NW>*>(LONG ? (void*)&U.s : (void*)&S_own);
    extern __shared__ __attribute__((aligned(16))) uint16_t s_sc[];  // scores (2 bytes a key of the cache, whole rows), then the selected rows
    __shared__ __attribute__((aligned(16))) uint32_t hist[NBR];
    __shared__ uint32_t s_codes[(G + 1) * WD];  // codes of the query heads and of the appended key
    __shared__ uint32_t s_tot[NW];
    __shared__ int s_T, s_lt;
    __shared__ int s_page[PAGED ? MAX_KEYS / 16 : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.x, b = blockIdx.y;
    const int64_t u = (int64_t)b * a.Hkv + h;
    const int hq0 = h * G;
    // what does not depend on the sequence length is requested first
    Hash hash;
    hash.fetch(a.W_H + (int64_t)h * HATA_D * R);
    const uint16_t* qv = a.q + ((int64_t)b * a.Hq + hq0) * HATA_D;
    typename Hash::Vector x[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p)
        if (4 * p < G) x[p] = Hash::fetch_x(qv + min(4 * p + (lane & 3), G - 1) * HATA_D);
    int my_page[PAGED ? MAX_KEYS / 16 / NT + 1 : 1] = {};
    if constexpr (PAGED)
#pragma unroll
        for (int i = 0; i < MAX_KEYS / 16 / NT + 1; ++i)
            if (tid + i * NT < min(a.pv.max_blocks, MAX_KEYS / 16)) my_page[i] = a.pv.table[(int64_t)b * a.pv.max_blocks + tid + i * NT];
    const int L = clampi(a.seq_len[b], 0, PAGED ? min(a.L_cap, a.pv.max_blocks << a.pv.shift) : a.L_cap);
    const int keff = min(clampi(a.kbud[b], 0, a.k_max), L);
    for (int i = tid; i < NBR; i += NT) hist[i] = 0;
    if (tid == 0) { s_T = 0; s_lt = 0; }
    if constexpr (PAGED) {  // where the pages' parts of this head start, in rows of the pools (fewer than 2^31: the host checks)
#pragma unroll
        for (int i = 0; i < MAX_KEYS / 16 / NT + 1; ++i)
            if (tid + i * NT < MAX_KEYS / 16) s_page[tid + i * NT] = (clampi(my_page[i], 0, a.pv.n_pages - 1) * a.Hkv + h) << a.pv.shift;
        __syncthreads();
    }
    auto cache_row = [&](int n) -> int64_t {
        if constexpr (PAGED) return (int64_t)(s_page[n >> a.pv.shift] + (n & ((1 << a.pv.shift) - 1)));
        else return u * a.L_cap + n;
    };
    const bool own = a.append && L > 0;  // row L - 1 is encoded here
    if (own) {
        const uint16_t* kx = PAGED ? a.K + cache_row(L - 1) * HATA_D : a.K + b * a.sb + h * a.sh + (int64_t)(L - 1) * a.sn;
        if (G % 4 == 0 || (lane & 3) == G % 4) x[PASSES - 1] = Hash::fetch_x(kx);
    }
    // the codes of this thread's keys, tid + 1024 j (row L - 1 is scored from the code computed here)
    const int stop = own ? L - 1 : L;
    struct Code { uint32_t w[WD]; } kc[UNR];
    auto load_codes = [&](int n0) {
#pragma unroll
        for (int j = 0; j < UNR; ++j) {
            const int n = n0 + NT * j;
            if (n < stop) {
                const uint32_t* cp = a.codes + cache_row(n) * WD;
                if constexpr (WD == 1) {
                    kc[j].w[0] = cp[0];
                } else if constexpr (WD == 2) {
                    const uint2 v = *reinterpret_cast<const uint2*>(cp);
                    kc[j].w[0] = v.x; kc[j].w[1] = v.y;
                } else {
#pragma unroll
                    for (int i = 0; i < WD / 4; ++i) {
                        typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
                        const uint4 v = LONG && WD == 4 ? __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(cp) + i))
                                                        : reinterpret_cast<const uint4*>(cp)[i];
                        kc[j].w[4 * i] = v.x; kc[j].w[4 * i + 1] = v.y; kc[j].w[4 * i + 2] = v.z; kc[j].w[4 * i + 3] = v.w;
                    }
                }
            }
        }
    };
    constexpr bool EARLY = WD <= 4;  // (at r = 256 the weights need the registers)
    if (EARLY) load_codes(tid);
    // ---- HashEncode(Q), HashEncode(K_new)
    const int vectors = own ? G + 1 : G, group = wave % Hash::GROUPS;
    double acc[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p)
        if (4 * p < G) acc[p] = hash.project(x[p]);
        else if (own) acc[p] = hash.project_one(x[p]);
    if constexpr (Hash::PARTS > 1) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (4 * p < G || own) U.part[p][wave][lane] = acc[p];
        __syncthreads();
        // the waves of a group of columns share the passes
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            if ((4 * p < G || own) && p % Hash::PARTS == wave / Hash::GROUPS) {
                double t = U.part[p][group][lane];
#pragma unroll
                for (int i = 1; i < Hash::PARTS; ++i) t += U.part[p][group + i * Hash::GROUPS][lane];
                if (4 * p < G) Hash::store_bits(t, s_codes, group, 4 * p, vectors);
                else Hash::store_bits_one(t, s_codes, group, G);
            }
        }
    } else {
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (4 * p < G) Hash::store_bits(acc[p], s_codes, group, 4 * p, vectors);
            else if (own) Hash::store_bits_one(acc[p], s_codes, group, G);
    }
    __syncthreads();
    if (tid < G * WD) a.qcodes[((int64_t)b * a.Hq + hq0) * WD + tid] = s_codes[tid];
    if (own && tid < WD) a.codes[cache_row(L - 1) * WD + tid] = s_codes[G * WD + tid];
    // query fragments for the attention
    uint32_t qr[MFMA ? 1 : G][4];
    uint4 qb[4];
    if constexpr (MFMA) attn_load_q_mfma<G>(qv, qb);
    else attn_load_q<G>(qv, qr);
    // ---- scores
    constexpr bool PLANES = HammingSum<WD, G>::PLANES;
    HammingSum<WD, G> dist;
    uint32_t qc[PLANES ? 1 : G][WD];
    if constexpr (PLANES) {
        dist.init(s_codes);
    } else {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int w = 0; w < WD; ++w) qc[g][w] = __builtin_amdgcn_readfirstlane(s_codes[g * WD + w]);
    }
    auto distance = [&](const uint32_t (&k)[WD]) {
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
    };
    auto scored = [&](int n, const uint32_t (&k)[WD]) {
        const uint32_t s = distance(k);
        if constexpr (LONG) {
            const int i = n & ((1 << a.log2_kpt) - 1), row = i >> 1;
            s_sc[2 * (row * NT + (((n >> a.log2_kpt) + 4 * row) & (NT - 1))) + (i & 1)] = (uint16_t)s;
        } else {
            s_sc[n] = (uint16_t)s;
        }
        atomicAdd(&hist[s], 1u);
    };
    // (one set of codes while the other is scored: no faster, a compute unit's own rate for its misses bounds a long stream)
    if (!EARLY) load_codes(tid);
    for (int n0 = tid;;) {
#pragma unroll
        for (int j = 0; j < UNR; ++j)
            if (n0 + NT * j < stop) scored(n0 + NT * j, kc[j].w);
        n0 += NT * UNR;
        if (!LONG || n0 - tid >= stop) break;
        load_codes(n0);
    }
    if (own && tid == NT - 1) {
        uint32_t kw[WD];
#pragma unroll
        for (int w = 0; w < WD; ++w) kw[w] = s_codes[G * WD + w];
        scored(L - 1, kw);
    }
    __syncthreads();
    // ---- threshold T: the smallest score whose count reaches keff; s_lt keys are below it
    {
        constexpr int SEG = NBR / 4 <= NT ? 4 : 8;  // consecutive scores of a thread
        static_assert(SEG * NT >= NBR, "a thread per segment");
        uint32_t c[SEG];
#pragma unroll
        for (int i = 0; i < SEG; i += 4) {
            uint4 v = make_uint4(0, 0, 0, 0);
            if (tid * SEG + i < NBR) v = *reinterpret_cast<const uint4*>(&hist[tid * SEG + i]);
            c[i] = v.x; c[i + 1] = v.y; c[i + 2] = v.z; c[i + 3] = v.w;
        }
        uint32_t loc = 0;
#pragma unroll
        for (int i = 0; i < SEG; ++i) loc += c[i];
        const uint32_t incl = wave_incl_scan(loc);
        if (lane == 63) s_tot[wave] = incl;
        __syncthreads();
        uint32_t all;
        uint32_t run = before_wave(s_tot, all) + incl - loc;
        if (run < (uint32_t)keff && run + loc >= (uint32_t)keff) {
            int T = tid * SEG;
#pragma unroll
            for (int i = 0; i < SEG; ++i) {
                if (run + c[i] < (uint32_t)keff) { run += c[i]; ++T; c[i] = 0; }
                else break;
            }
            s_T = T;
            s_lt = (int)run;
        }
        __syncthreads();
    }
    // ---- ordered compaction: a thread takes KPT consecutive keys; ties go to the lowest rows
    int32_t* io = a.idx + u * a.k_max;
    for (int p = keff + tid; p < a.k_max; p += NT) io[p] = -1;
    {
        const int T = s_T, need = keff - s_lt;
        constexpr int MAX_KPT = MAX_KEYS / NT;
        const int kpt = LONG ? 1 << a.log2_kpt : MAX_KPT, n0 = tid * kpt;
        uint32_t m_lt = 0, m_eq = 0;  // bit i: key n0 + i is below / at the threshold
        uint32_t sv[MAX_KPT / 2];     // two scores each
#pragma unroll
        for (int w = 0; w < MAX_KPT / 2; ++w) {
            sv[w] = 0;
            if (!LONG || 2 * w < kpt) {
                const uint32_t v = sv[w] = reinterpret_cast<const uint32_t*>(s_sc)[LONG ? w * NT + ((tid + 4 * w) & (NT - 1)) : tid * (MAX_KPT / 2) + w];
                const int s0 = (int)(v & 0xffffu), s1 = (int)(v >> 16);
                m_lt |= (s0 < T ? 1u : 0u) << (2 * w) | (s1 < T ? 2u : 0u) << (2 * w);
                m_eq |= (s0 == T ? 1u : 0u) << (2 * w) | (s1 == T ? 2u : 0u) << (2 * w);
            }
        }
        // The scores, where they are wanted: from here, many of a thread's at a time, as stores of two bytes a key between the loads
        // of the codes are waited for with them (r = 128, 16 sequences of eight KV heads, 16384 keys each 28.9 -> 25.6 us a layer, one of
        // them that long and the others of 500 26.2 -> 23.6).
        if (a.scores && n0 < L) {
            uint16_t* const sp = a.scores + u * a.L_cap + n0;
            constexpr int STEP = LONG ? 8 : 4;  // (kpt is a multiple)
            const bool whole = (reinterpret_cast<uintptr_t>(sp) & (2 * STEP - 1)) == 0;
#pragma unroll
            for (int i = 0; i < MAX_KPT; i += STEP) {
                if (whole && i < kpt && n0 + i + STEP <= L) {
                    if constexpr (LONG) *reinterpret_cast<uint4*>(sp + i) = make_uint4(sv[i / 2], sv[i / 2 + 1], sv[i / 2 + 2], sv[i / 2 + 3]);
                    else *reinterpret_cast<uint2*>(sp + i) = make_uint2(sv[i / 2], sv[i / 2 + 1]);
                } else if (i < kpt) {
#pragma unroll
                    for (int e = i; e < i + STEP; ++e)
                        if (n0 + e < L) sp[e] = (uint16_t)(sv[e / 2] >> (e % 2 * 16));
                }
            }
        }
        const int n_live = keff > 0 ? clampi(L - n0, 0, kpt) : 0;
        const uint32_t live = (1u << n_live) - 1u;  // (at most 16 keys)
        m_lt &= live;
        m_eq &= live;
        const uint32_t mine = __popc(m_lt) | (__popc(m_eq) << 16);  // (at most 16384 keys: both halves' sums fit)
        const uint32_t incl = wave_incl_scan(mine);
        if (lane == 63) s_tot[wave] = incl;
        __syncthreads();  // (every thread has read its scores: s_sc becomes the row list)
        uint32_t all;
        const uint32_t before = before_wave(s_tot, all) + incl - mine;
        const int lt_b = (int)(before & 0xffffu), eq_b = (int)(before >> 16);
        // of this thread's keys at the threshold the first ones, as many as the threads before leave
        const int ties_before = min(eq_b, need);
        uint32_t keep = m_eq;
        const int avail = min((int)__popc(m_eq), need - ties_before);
        while ((int)__popc(keep) > avail) keep &= ~(0x80000000u >> __clz(keep));  // drop the highest row
        uint32_t sel = m_lt | keep;
        int r = lt_b + ties_before;
        while (sel) {  // (a thread holds k / L of its keys on average)
            const int n = n0 + __ffs(sel) - 1;
            sel &= sel - 1;
            s_sc[r] = (uint16_t)n;
            io[r] = n;
            ++r;
        }
    }
    __syncthreads();
    // ---- attention over the selected rows
    if constexpr (PAGED) {
        auto row_of = [&](int row) { return (int)cache_row((int)s_sc[row]); };
        const int rows = (a.pv.n_pages * a.Hkv) << a.pv.shift;
        if constexpr (MFMA) attn_rows_mfma<G, NW, LONG>(qb, a.K, a.V, HATA_D, rows, 0, keff, a.scale_log2, row_of, S, U.vt);
        else attn_rows<G, 4, NW>(qr, a.K, a.V, HATA_D, rows, 0, keff, a.scale_log2, row_of, S);
    } else {
        const uint16_t* Kb = a.K + b * a.sb + h * a.sh;
        const uint16_t* Vb = a.V + b * a.sb + h * a.sh;
        auto row_of = [&](int row) { return (int)s_sc[row]; };
        if constexpr (MFMA) attn_rows_mfma<G, NW, LONG>(qb, Kb, Vb, a.sn, a.L_cap, 0, keff, a.scale_log2, row_of, S, U.vt);
        else attn_rows<G, 4, NW>(qr, Kb, Vb, a.sn, a.L_cap, 0, keff, a.scale_log2, row_of, S);
    }
    // ---- the waves' states together: a thread per (head, channel)
    for (int i = tid; i < G * HATA_D; i += NT) {
        const int g = i / HATA_D, ch = i % HATA_D;
        float m[NW], M = HATA_NEG_INF;
#pragma unroll
        for (int w = 0; w < NW; ++w) { m[w] = S.m[w][g]; M = fmaxf(M, m[w]); }
        float av = 0.f, l = 0.f;
        if (M != HATA_NEG_INF) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float f = fast_exp2(m[w] - M);
                av = fmaf(f, S.acc[w][g][ch], av);
                l = fmaf(f, S.l[w][g], l);
            }
        }
        const float o = l > 0.f ? av / l : 0.f;
        const int64_t at = ((int64_t)b * a.Hq + hq0) * HATA_D + i;
        a.out[at] = (uint16_t)f32_to_bf16(o);
        if (a.out_f32) a.out_f32[at] = o;
    }
}

template <int WD, int G>
static const void* unit_fn_g(bool paged, bool lng) {
    if (paged) return lng ? (const void*)&decode_step_unit_kernel<WD, G, true, true> : (const void*)&decode_step_unit_kernel<WD, G, true, false>;
    return lng ? (const void*)&decode_step_unit_kernel<WD, G, false, true> : (const void*)&decode_step_unit_kernel<WD, G, false, false>;
}
template <int WD>
static const void* unit_fn(int G, bool paged, bool lng) {
    switch (G) {
        case 1: return unit_fn_g<WD, 1>(paged, lng);
        case 2: return unit_fn_g<WD, 2>(paged, lng);
        case 4: return unit_fn_g<WD, 4>(paged, lng);
        case 5: return unit_fn_g<WD, 5>(paged, lng);
        case 8: return unit_fn_g<WD, 8>(paged, lng);
        default: return nullptr;
    }
}
static const void* unit_kernel_for(int Wd, int G, bool paged, bool lng) {
    switch (Wd) {
        case 1: return unit_fn<1>(G, paged, lng);
        case 2: return unit_fn<2>(G, paged, lng);
        case 4: return unit_fn<4>(G, paged, lng);
        case 8: return unit_fn<8>(G, paged, lng);
        default: return nullptr;
    }
}
// consecutive keys of a thread, as a power of two
static int unit_log2_kpt(int L_cap) {
    int l = 2;
    while ((HATA_UNIT_THREADS << l) < L_cap) ++l;
    return l;
}

hipError_t prepare_unit_step(hata_ctx* c) {
    c->unit_keys = 0;
    if (c->cfg.L_cap > HATA_UNIT_KEYS_LONG || !unit_kernel_for(c->Wd, c->G, false, false)) return hipSuccess;
    c->unit_keys = HATA_UNIT_THREADS << unit_log2_kpt(c->cfg.L_cap);
    const bool lng = c->unit_keys > HATA_UNIT_KEYS;
    for (int paged = 0; paged < 2; ++paged) {  // (the kernel's limit, not this context's size)
        const hipError_t e = hipFuncSetAttribute(unit_kernel_for(c->Wd, c->G, paged != 0, lng), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (lng ? HATA_UNIT_KEYS_LONG : HATA_UNIT_KEYS) * 2);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_unit_step(const hata_ctx* c, const void* q, const void* K, const void* V, const float* W_H, uint32_t* codes,
                            int append, const int32_t* seq_len, const int32_t* k, int B, float sm_scale, void* out,
                            float* out_f32, hipStream_t s, const PageView* pages) {
    const hata_config& f = c->cfg;
    UnitArgs a;
    a.log2_kpt = unit_log2_kpt(f.L_cap);
    a.q = (const uint16_t*)q; a.K = (const uint16_t*)K; a.V = (const uint16_t*)V; a.W_H = W_H;
    a.seq_len = seq_len; a.kbud = k; a.codes = codes; a.qcodes = c->qcodes;
    // a shared device's contiguous cache takes two or three launches for any other shape, and these always leave the scores in the workspace
    a.scores = c->keep_scores || (!pages && c->step_mode == 3) ? c->scores : nullptr;
    a.idx = c->idx; a.out = (uint16_t*)out; a.out_f32 = out_f32;
    a.Hq = f.Hq; a.Hkv = f.Hkv; a.L_cap = f.L_cap; a.k_max = f.k_max; a.append = append;
    a.sb = f.kv_stride_b; a.sh = f.kv_stride_h; a.sn = f.kv_stride_n;
    a.scale_log2 = sm_scale * 1.4426950408889634f;
    a.pv = pages ? *pages : PageView{nullptr, 0, 0, 0};
    void* args[] = {(void*)&a};
    return hipLaunchKernel(unit_kernel_for(c->Wd, c->G, pages != nullptr, c->unit_keys > HATA_UNIT_KEYS), dim3(f.Hkv, B), dim3(HATA_UNIT_THREADS), args,
                           (size_t)c->unit_keys * 2, s);
}

}  // namespace hata
