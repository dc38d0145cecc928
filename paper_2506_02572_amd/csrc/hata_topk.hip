// Stand-alone selection (Alg. 3 of the paper: Idx = TopK(S, N)) for scores that are already stored: a counting
// select over the <= G*r + 1 score values with ordered compaction, lower row first on equal scores.
//   topk_unit_kernel               one workgroup per (sequence, KV head) unit, caches of up to 65536 rows
//   hist_kernel + compact_kernel   longer caches: chunk histograms and, by the last workgroup of each unit, the
//                                  unit threshold; then the compaction
#include <type_traits>
#include "hata_device.h"
#include "hata_internal.h"
#include "hata_select.h"

namespace hata {

// grid = (n_chunks, Hkv, B), 256 threads: histogram of one chunk of stored scores; the last workgroup
// of a unit to finish goes on to the unit's threshold and chunk offsets (finish_unit).
__global__ __launch_bounds__(256) void hist_kernel(
    const uint16_t* __restrict__ scores, const int32_t* __restrict__ seq_len,
    const int32_t* __restrict__ kbud, uint16_t* __restrict__ chunk_hist, int Hkv, int L_cap, int k_max,
    int chunk, int n_chunks, int NB, int NBP, int32_t* __restrict__ chunk_info,
    int32_t* __restrict__ unit_info, uint32_t* __restrict__ unit_counter, uint32_t* __restrict__ unit_hist) {
    extern __shared__ uint32_t hist[];
    __shared__ ThresholdLds S;
    __shared__ int last_flag;
    const int tid = threadIdx.x;
    const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int L = clampi(seq_len[b], 0, L_cap);
    const int base = c * chunk;
    const int64_t u = (int64_t)b * Hkv + h;
    if (base >= L) {
        if (L == 0 && c == 0 && tid == 0) {  // empty sequence: nothing selected
            unit_info[u * 2 + 0] = 0;
            unit_info[u * 2 + 1] = 0;
            chunk_info[u * (n_chunks + 1) * 2 + 0] = 0;
            chunk_info[u * (n_chunks + 1) * 2 + 1] = 0;
        }
        return;
    }
    const int end = min(base + chunk, L);
    for (int i = tid; i < NB; i += 256) hist[i] = 0;
    __syncthreads();
    const uint16_t* sp = scores + u * L_cap;
    for (int n = base + tid; n < end; n += 256) atomicAdd(&hist[min((int)sp[n], NB - 1)], 1u);
    __syncthreads();
    write_chunk_hist(chunk_hist + (u * n_chunks + c) * NBP, hist, NB, NBP);
    const int keff = min(clampi(kbud[b], 0, k_max), L);
    finish_unit(u, (L + chunk - 1) / chunk, keff, chunk_hist + u * n_chunks * NBP, NB, NBP, n_chunks, chunk_info,
                unit_info, unit_counter, unit_hist, hist, S, &last_flag);
}

// grid = (n_chunks, Hkv, B), 256 threads: ordered compaction of one chunk into the index list.
__global__ __launch_bounds__(256) void compact_kernel(
    const uint16_t* __restrict__ scores, const int32_t* __restrict__ seq_len,
    const int32_t* __restrict__ chunk_info, const int32_t* __restrict__ unit_info,
    int32_t* __restrict__ idx, int Hkv, int L_cap, int k_max, int chunk, int n_chunks) {
    __shared__ uint32_t scan4[4];
    const int tid = threadIdx.x;
    const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int L = clampi(seq_len[b], 0, L_cap);
    const int64_t u = (int64_t)b * Hkv + h;
    const int T = unit_info[u * 2 + 0];
    const int keff = unit_info[u * 2 + 1];
    int32_t* out = idx + u * k_max;
    if (c == 0)  // pad the row
        for (int i = keff + tid; i < k_max; i += 256) out[i] = -1;
    const int base = c * chunk;
    if (base >= L) return;
    const int32_t* ci = chunk_info + (u * (n_chunks + 1) + c) * 2;
    const int off = ci[0], take = ci[1];
    if (ci[2] == off) return;  // nothing selected in this chunk
    const uint16_t* sp = scores + u * L_cap;
    const int end = min(base + chunk, L);
    compact_chunk_any(chunk / 256, sp, base, end, T, off, take, scan4,
                      [&](int pos, int n) { if (pos < k_max) out[pos] = n; });
}

// One workgroup of 1024 threads per unit: its scores are staged in LDS once, thread t owns the 8 NV consecutive
// keys of the aligned 16-byte words NV t .. NV t + NV - 1, and the histogram, the threshold and the ranks never
// leave the workgroup.  grid = (Hkv, B).  Bound by one compute unit's instructions per key, so every pass over all
// keys compares two at a time with packed 16-bit instructions into one mask per thread, and only the few keys a
// mask names are handled singly: with NV > 1 a histogram of one pair of keys per thread gives a score below which
// about twice the budget lies, and only keys up to that score are counted (should they be fewer than the budget
// after all, everything is).  Two launches with hand-offs through memory took 18.6 us at 64 units of 17003 keys
// and 22.6 us of 65000, this takes 7.4 and 12.1.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

template <int NV>
__global__ __launch_bounds__(1024) void topk_unit_kernel(const uint16_t* __restrict__ scores,
                                                         const int32_t* __restrict__ seq_len,
                                                         const int32_t* __restrict__ kbud, int32_t* __restrict__ idx,
                                                         int Hkv, int L_cap, int k_max, int NB, int64_t n_scores) {
    using Mask = std::conditional_t<(NV > 4), uint64_t, uint32_t>;  // one bit per key of the thread
    extern __shared__ __attribute__((aligned(16))) uint16_t sc[];   // [NV * 8192] scores
    __shared__ uint32_t s_tot[16];                                  // per wave
    __shared__ int s_T, s_need;
    uint32_t* hist = reinterpret_cast<uint32_t*>(sc + NV * 8192);  // [NB]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = blockIdx.x, b = blockIdx.y;
    const int64_t u = (int64_t)b * Hkv + h;
    const int L = clampi(seq_len[b], 0, L_cap);
    const int keff = min(clampi(kbud[b], 0, k_max), L);
    const uint16_t* sp = scores + u * L_cap;
    int32_t* out = idx + u * k_max;
    const int shift = (int)((reinterpret_cast<uintptr_t>(sp) & 15) / 2);  // keys before the unit's in its first word
    {
        // whole words of the array first (loads without a branch between them, so that all are in flight
        // together), then those that reach over an end of it; keys outside the unit are masked below
        uint4 v[NV];
        const uint4* words = reinterpret_cast<const uint4*>(sp - shift);
        const int first = u * L_cap < shift ? 1 : 0;
        const int last = (int)min((n_scores - u * L_cap + shift) / 8, (int64_t)((L + shift + 7) / 8)) - 1;
        if (last >= first) {
#pragma unroll
            for (int j = 0; j < NV; ++j) v[j] = words[clampi(j * 1024 + tid, first, last)];
#pragma unroll
            for (int j = 0; j < NV; ++j) reinterpret_cast<uint4*>(sc)[j * 1024 + tid] = v[j];
        }
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int w = j * 1024 + tid, n = w * 8 - shift;
            if (n < L && (w < first || w > last)) {
#pragma unroll
                for (int i = 0; i < 8; ++i) sc[w * 8 + i] = n + i >= 0 && n + i < L ? sp[n + i] : (uint16_t)0;
            }
        }
    }
    for (int i = keff + tid; i < k_max; i += 1024) out[i] = -1;
    if (keff == 0) return;
    for (int i = tid; i < NB; i += 1024) hist[i] = 0;
    if (tid == 0) s_T = NB - 1;
    const int own = tid * NV * 8, n0 = own - shift;  // first key of the thread: in sc, in the unit
    const int dead_lo = clampi(-n0, 0, NV * 8), dead_hi = NV * 8 - clampi(L - n0, 0, NV * 8);
    Mask live = dead_hi < NV * 8 ? (Mask)(~(Mask)0) >> (sizeof(Mask) * 8 - NV * 8 + dead_hi) : (Mask)0;
    live &= dead_lo < NV * 8 ? (Mask)(~(Mask)0) << dead_lo : (Mask)0;
    __syncthreads();
    // scores above the largest value count as the largest
    auto score = [&](int i) { return min((int)sc[own + i], NB - 1); };
    // the thread's keys with a score <= t
    auto up_to = [&](int t) {
        Mask m = 0;
        const u16x2 t1 = {(uint16_t)(t + 1), (uint16_t)(t + 1)}, one = {1, 1};
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int w = (j + tid) % NV;  // (no two lanes of a phase on the same banks)
            const uint4 v = reinterpret_cast<const uint4*>(sc)[tid * NV + w];
            const uint32_t d[4] = {v.x, v.y, v.z, v.w};
            uint32_t x = 0;  // key 2 i in bit 2 i, key 2 i + 1 in bit 16 + 2 i
#pragma unroll
            for (int i = 0; i < 4; ++i)
                x |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_elementwise_sub_sat(t1, __builtin_bit_cast(u16x2, d[i])), one)) << (2 * i);
            m |= (Mask)((x | (x >> 15)) & 0xffu) << (8 * w);
        }
        return (Mask)(t >= NB - 1 ? live : m & live);
    };
    auto count = [&](Mask m) {
        while (m) {
            const int i = NV > 4 ? __ffsll((unsigned long long)m) - 1 : __ffs((uint32_t)m) - 1;
            m &= m - 1;
            atomicAdd(&hist[score(i)], 1u);
        }
    };
    // smallest score whose inclusive count reaches `want` -> s_T, want minus the keys below it -> s_need (both
    // left alone if none does); returns the number of keys counted.  Ends with the histogram clear.
    auto search = [&](int want) {
        __syncthreads();
        const int seg = (NB + 1023) / 1024, s0 = tid * seg;  // (at most five bins a thread)
        uint32_t x[5], loc = 0;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            x[i] = i < seg && s0 + i < NB ? hist[s0 + i] : 0u;
            if (x[i]) hist[s0 + i] = 0;
            loc += x[i];
        }
        const uint32_t incl = wave_incl_scan(loc);
        if (lane == 63) s_tot[wave] = incl;
        __syncthreads();
        const uint32_t scan = wave_incl_scan(lane < 16 ? s_tot[lane] : 0u);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)scan, 15);
        uint32_t run = incl - loc + (wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)scan, wave - 1) : 0u);
        if (run < (uint32_t)want && run + loc >= (uint32_t)want) {
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                if (run < (uint32_t)want && run + x[i] >= (uint32_t)want) { s_T = s0 + i; s_need = want - (int)run; }
                run += x[i];
            }
        }
        __syncthreads();
        return (int)total;
    };
    int most = NB - 1;
    if constexpr (NV > 1) {
        count(live & (Mask)3);  // one pair of keys per thread
        search(keff / (4 * NV) * 2 + 64);
        most = s_T;
    }
    Mask low = up_to(most);
    count(low);
    if (search(keff) < keff) {
        low = live;
        count(low);
        search(keff);
    }
    const int T = s_T, need = s_need;
    Mask m_lt = 0, ties = 0;
    while (low) {
        const Mask rest = low & (low - 1), bit = low ^ rest;
        const int x = score(NV > 4 ? __ffsll((unsigned long long)low) - 1 : __ffs((uint32_t)low) - 1);
        m_lt |= x < T ? bit : (Mask)0;
        ties |= x == T ? bit : (Mask)0;
        low = rest;
    }
    const int lt = NV > 4 ? __popcll(m_lt) : __popc((uint32_t)m_lt), eq = NV > 4 ? __popcll(ties) : __popc((uint32_t)ties);
    const uint32_t mine = (uint32_t)lt | ((uint32_t)eq << 16);  // (no exclusive prefix of either count reaches 65536)
    const uint32_t incl = wave_incl_scan(mine);
    if (lane == 63) s_tot[wave] = incl;
    __syncthreads();
    const uint32_t scan = wave_incl_scan(lane < 16 ? s_tot[lane] : 0u);
    const uint32_t before = incl - mine + (wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)scan, wave - 1) : 0u);
    // ties go to the lowest rows
    const int ties_before = min((int)(before >> 16), need);
    for (int drop = eq - min(eq, need - ties_before); drop > 0; --drop)
        ties &= ~((Mask)1 << (NV > 4 ? 63 - __clzll((unsigned long long)ties) : 31 - __clz((uint32_t)ties)));
    int pos = (int)(before & 0xffffu) + ties_before;
    for (Mask m = m_lt | ties; m; m &= m - 1, ++pos)
        if (pos < keff) out[pos] = n0 + (NV > 4 ? __ffsll((unsigned long long)m) : __ffs((uint32_t)m)) - 1;
}

static size_t topk_unit_lds(int NB, int nv) { return (size_t)nv * 16384 + (size_t)NB * 4; }

// (more than 64 KB of dynamic LDS has to be asked for: what the largest number of score values takes, since the limit
// belongs to the kernel and every context sets it)
hipError_t prepare_topk() {
    hipError_t e = hipFuncSetAttribute((const void*)topk_unit_kernel<4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)topk_unit_lds(HATA_MAX_NB, 4));
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void*)topk_unit_kernel<8>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)topk_unit_lds(HATA_MAX_NB, 8));
}

hipError_t launch_topk(const hata_ctx* c, const uint16_t* scores, const int32_t* seq_len,
                       const int32_t* k, int B, int32_t* idx, hipStream_t s) {
    const hata_config& f = c->cfg;
    // words per thread: a unit may begin inside a word
    const int shift = f.L_cap % 8 ? 7 : (int)((reinterpret_cast<uintptr_t>(scores) & 15) / 2);
    const int words = (f.L_cap + shift + 8191) / 8192;
    if (words <= 8) {  // (the scores fit in LDS)
#define HATA_LAUNCH_UNIT(NV)                                                                                      \
    hipLaunchKernelGGL((topk_unit_kernel<NV>), dim3(f.Hkv, B), dim3(1024), topk_unit_lds(c->NB, NV), s, scores, seq_len, \
                       k, idx, f.Hkv, f.L_cap, f.k_max, c->NB, (int64_t)B * f.Hkv * f.L_cap)
        if (words <= 1) HATA_LAUNCH_UNIT(1);
        else if (words <= 2) HATA_LAUNCH_UNIT(2);
        else if (words <= 4) HATA_LAUNCH_UNIT(4);
        else HATA_LAUNCH_UNIT(8);
#undef HATA_LAUNCH_UNIT
        return hipGetLastError();
    }
    const dim3 grid(c->n_chunks, f.Hkv, B);
    const size_t lds = (size_t)c->NB * 4;
    hipLaunchKernelGGL(hist_kernel, grid, dim3(256), lds, s, scores, seq_len, k, c->chunk_hist,
                       f.Hkv, f.L_cap, f.k_max, c->chunk, c->n_chunks, c->NB, c->NBP, c->chunk_info,
                       c->unit_info, c->unit_counter, c->unit_hist);
    hipLaunchKernelGGL(compact_kernel, grid, dim3(256), 0, s, scores, seq_len, c->chunk_info,
                       c->unit_info, idx, f.Hkv, f.L_cap, f.k_max, c->chunk, c->n_chunks);
    return hipGetLastError();
}

}  // namespace hata
