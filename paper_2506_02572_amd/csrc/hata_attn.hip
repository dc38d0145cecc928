// Decode attention over a list of cache rows (Alg. 3 of the paper: Gather + Attention, with
// the gather fused into the attention kernel; Eq. 2 third line, scale of Eq. 1).
//
// One kernel template, two row sources:
//   ROWS_IDX     rows come from an index list in memory            (hata_sparse_decode)
//   ROWS_SELECT  the rows of one chunk of the cache (a few, of a very long one) that the unit
//                threshold selects: ordered compaction of the chunk's stored scores; its part of
//                the index list is written as a by-product  (hata_decode_step, three-launch form)
//
// Split over the rows: every workgroup handles a slice of a unit's rows for HT query heads of
// the group at once (each K/V row is read once for all of them), keeps an online-softmax
// state per wave, and writes one partial (max, sum, weighted V) per query head; the last
// workgroup of a (unit, head tile) to finish merges the partials and writes the output, so no
// separate merge launch is needed.  A row is 256 B = 16 lanes x 128-bit, so a wave reads
// four whole rows per load instruction.  bf16 inputs, fp32 softmax and accumulation.
#include "hata_device.h"
#include "hata_internal.h"
#include "hata_select.h"
#include "hata_attn_core.h"

namespace hata {

enum { ROWS_IDX = 0, ROWS_SELECT = 2 };

struct AttnArgs {
    const uint16_t* q;
    const uint16_t* K;
    const uint16_t* V;
    const int32_t* idx_in;      // ROWS_IDX
    int32_t* idx_out;           // ROWS_SELECT
    const int32_t* count_src;   // ROWS_IDX: k[B]
    const uint16_t* scores;     // ROWS_SELECT ...
    const int32_t* seq_len;
    const int32_t* chunk_info;
    const int32_t* unit_info;
    int chunk, n_chunks, chunks_per_split, owners, piece_rows, B;  // (chunk, chunks_per_split: powers of two)
    float* partials;
    uint32_t* counter;
    int counter_stride;
    uint16_t* out;
    float* out_f32;
    int Hq, Hkv, G, L_cap, k_max, rows_per_wg, n_splits;
    int64_t sb, sh, sn;
    float scale_log2;
};

// grid = (splits, Hkv * (G / HT), B), in ROWS_SELECT (owners, .., B + layers for the further pieces); 256 threads.
// ROWS_SELECT: the first `owners` splits are a chunk each (or as many as leave at most 256 splits to merge), so that
// everything the selection needs -- the chunk's scores, its offset and ties, the threshold -- is at addresses known from
// the start, and on the XCD that scored the chunk.  Slices of the index list instead, which had to find their chunks first,
// took 18.4 us per launch at 16 units of 20011 keys, this takes 10.4.  A prompt's selected rows may all lie in a chunk or
// two, though: an owner attends over the first piece_rows rows of its chunk only, and the further pieces go to the splits
// behind the owners, which compact that chunk again: 8 units of 131072 keys, 2048 rows all in one place, 64.5 -> 35.0 us a step
// (31.0 where they are spread, and those splits return at once; 30.6 without them).
template <int HT, int MODE>
__global__ __launch_bounds__(256) void attn_kernel(const AttnArgs a) {
    constexpr bool MFMA = HT >= 4;  // matrix-core form of the attention core
    __shared__ __attribute__((aligned(16))) AttnLds<HT> S;
    __shared__ __attribute__((aligned(16))) uint16_t s_vt[MFMA ? HATA_VT_ELEMS : 8];
    extern __shared__ __attribute__((aligned(16))) uint16_t s_sc[];  // ROWS_SELECT: the chunk's scores, then its selected rows
    __shared__ uint32_t scan4[4];
    __shared__ int s_last;
    const int tid = threadIdx.x;
    const int tiles = a.G / HT;
    const int h = blockIdx.y / tiles;
    const int ht = blockIdx.y % tiles;
    int split = blockIdx.x, b = blockIdx.z;
    if (MODE == ROWS_SELECT && b >= a.B) {
        const int i = (b - a.B) * a.owners + split, further = a.n_splits - a.owners;
        b = i / further;
        if (b >= a.B) return;
        split = a.owners + (i + blockIdx.y) % further;
    }
    const int64_t u = (int64_t)b * a.Hkv + h;
    const int hq0 = h * a.G + ht * HT;
    uint16_t* outp = a.out + ((int64_t)b * a.Hq + hq0) * HATA_D;
    float* outp32 = a.out_f32 ? a.out_f32 + ((int64_t)b * a.Hq + hq0) * HATA_D : nullptr;
    const uint16_t* Kb = a.K + b * a.sb + h * a.sh;
    const uint16_t* Vb = a.V + b * a.sb + h * a.sh;
    // query fragments first: nothing below depends on them until the rows are known
    uint32_t qr[MFMA ? 1 : HT][4];
    uint4 qb[4];
    if constexpr (MFMA) attn_load_q_mfma<HT>(a.q + ((int64_t)b * a.Hq + hq0) * HATA_D, qb);
    else attn_load_q<HT>(a.q + ((int64_t)b * a.Hq + hq0) * HATA_D, qr);
    auto zero_output = [&]() {
        for (int i = tid; i < HT * HATA_D; i += 256) {
            outp[i] = 0;
            if (outp32) outp32[i] = 0.f;
        }
    };
    int ns, slot = split;  // workgroups that contribute, this one's place among their partial results
    auto attend = [&](int row_begin, int row_end, auto row_of) {
        if constexpr (MFMA)
            attn_rows_mfma<HT>(qb, Kb, Vb, a.sn, a.L_cap, row_begin, row_end, a.scale_log2, row_of, S, s_vt);
        else
            attn_rows<HT, 4>(qr, Kb, Vb, a.sn, a.L_cap, row_begin, row_end, a.scale_log2, row_of, S);
    };
    if constexpr (MODE == ROWS_SELECT) {
        // what an owner reads is requested together: no address depends on the sequence's length
        const int per = a.chunks_per_split, span = per * a.chunk;
        const int32_t* ci_unit = a.chunk_info + u * (a.n_chunks + 1) * 2;
        auto entry = [&](int s) { return ci_unit + 2 * min(s * per, a.n_chunks); };
        const int seq = a.seq_len[b], T = a.unit_info[u * 2 + 0], budget = a.unit_info[u * 2 + 1];
        int off = 0, take = 0, next = 0;
        if (split < a.owners) {
            off = entry(split)[0];
            take = entry(split)[1];
            next = entry(split + 1)[0];
        }
        const int lane = tid & 63;
        const int first0 = *entry(lane), next0 = *entry(lane + 1);
        const int L = clampi(seq, 0, a.L_cap), keff = clampi(budget, 0, a.k_max);
        const int nc = (L + a.chunk - 1) >> __builtin_ctz(a.chunk);  // (entry nc closes the list: keff)
        const int live = (L + span - 1) >> __builtin_ctz(span);      // owners with keys
        int32_t* io = a.idx_out + u * a.k_max;
        if (split == 0) {
            if (ht == 0)  // slots of the index list past the selected count hold -1
                for (int p = keff + tid; p < a.k_max; p += 256) io[p] = -1;
            if (L == 0) zero_output();
        }
        auto selected = [&](int s, int first, int next) {
            return clampi(next - first, 0, min(min(span, L - s * span), a.k_max - clampi(first, 0, a.k_max)));
        };
        // pieces beyond an owner's first: lane l looks at owners l, l + 64, ... (the first of them are requested above);
        // returns how many there are, and where number `nth` of them is
        const float half_inv = 0.5f * __builtin_amdgcn_rcpf((float)a.piece_rows);  // (rows - 1) / piece_rows, exact below 2^20
        auto further_pieces = [&](int nth, int& own, int& piece) {
            int extra = 0;
            for (int s0 = 0; s0 < live; s0 += 64) {
                const int s = s0 + lane;
                const int first = s0 == 0 ? first0 : *entry(s);
                const int next = (s + 1) * per > nc ? keff : s0 == 0 ? next0 : *entry(s + 1);
                const int rows = s < live ? selected(s, first, next) : 0;
                const int more = rows > 0 ? (int)((float)(2 * rows - 1) * half_inv) : 0;
                if (__builtin_amdgcn_ballot_w64(more > 0) == 0) continue;
                const int upto = extra + (int)wave_incl_scan((uint32_t)more);
                const unsigned long long past = __builtin_amdgcn_ballot_w64(extra <= nth && upto > nth);
                if (past) {
                    const int l = __ffsll(past) - 1;
                    own = s0 + l;
                    piece = nth - __builtin_amdgcn_readlane(upto - more, l) + 1;
                }
                extra = __builtin_amdgcn_readlane(upto, 63);
            }
            return min(extra, a.n_splits - a.owners);
        };
        int own = split, piece = 0, extra = 0;
        if (split >= a.owners) {
            extra = further_pieces(split - a.owners, own, piece);
            if (split - a.owners >= extra) return;
            own = __builtin_amdgcn_readfirstlane(own);
            piece = __builtin_amdgcn_readfirstlane(piece);
            slot = live + split - a.owners;
            off = entry(own)[0];
            take = entry(own)[1];
            next = entry(own + 1)[0];
        } else if (split >= live) {
            return;
        }
        const int c0 = own * per, base = own * span, n_keys = min(span, L - base);
        if (c0 + per > nc) next = keff;
        // ties are granted in cache order, so those of consecutive chunks add up
        for (int i = 1; i < min(per, nc - c0); ++i) take += ci_unit[2 * (c0 + i) + 1];
        const uint16_t* sp = a.scores + u * a.L_cap + base;
        const bool whole = (reinterpret_cast<uintptr_t>(sp) & 15) == 0;
        for (int i = tid * 8; i < n_keys; i += 256 * 8) {
            if (whole && i + 8 <= n_keys) {
                *reinterpret_cast<uint4*>(&s_sc[i]) = *reinterpret_cast<const uint4*>(sp + i);
            } else {
                for (int e = i; e < min(i + 8, n_keys); ++e) s_sc[e] = sp[e];
            }
        }
        __syncthreads();
        const int cnt = selected(own, off, next);
        if (cnt > 0)  // (the same for the whole workgroup)
            compact_lds(s_sc, n_keys, span / 256, T, take, cnt, scan4, [&](int r, int n) {
                s_sc[r] = (uint16_t)n;
                if (ht == 0 && piece == 0) io[off + r] = base + n;
            });
        __syncthreads();
        attend(piece * a.piece_rows, min(cnt, (piece + 1) * a.piece_rows), [&](int row) { return base + (int)s_sc[row]; });
        if (piece == 0) extra = further_pieces(-1, own, piece);
        ns = live + extra;
    } else {
        const int count = clampi(a.count_src[b], 0, a.k_max);
        const int row_begin = split * a.rows_per_wg;
        if (row_begin >= count) {
            if (count == 0 && split == 0) zero_output();  // no row at all
            return;
        }
        const int row_end = min(row_begin + a.rows_per_wg, count);
        const int32_t* ip = a.idx_in + u * a.k_max;
        attend(row_begin, row_end, [&](int row) { return (int)ip[row]; });
        ns = (count + a.rows_per_wg - 1) / a.rows_per_wg;
    }
    const int64_t head_stride = (int64_t)a.n_splits * HATA_PSTRIDE;
    float* part0 = a.partials + ((int64_t)b * a.Hq + hq0) * head_stride;
    attn_emit<HT>(S, ns == 1, outp, outp32, part0 + (int64_t)slot * HATA_PSTRIDE, head_stride);
    if (ns == 1) return;
    // count the finished slices; the last workgroup merges them (partials are written with
    // write-through stores and read back with device-coherent loads)
    wait_stores();
    __syncthreads();
    if (tid == 0) {
        uint32_t* cnt = a.counter + (u * tiles + ht) * a.counter_stride;
        const uint32_t done = atomicAdd(cnt, 1u);
        const int last = (done == (uint32_t)(ns - 1));
        if (last) *cnt = 0;
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    attn_merge<HT>(S, part0, head_stride, ns, outp, outp32);
}

template <int HT>
static void launch_mode(int mode, const AttnArgs& a, dim3 grid, hipStream_t s) {
    const size_t lds = mode == ROWS_SELECT ? (size_t)a.chunk * a.chunks_per_split * 2 + 32 : 0;
    switch (mode) {
        case ROWS_SELECT: hipLaunchKernelGGL((attn_kernel<HT, ROWS_SELECT>), grid, dim3(256), lds, s, a); break;
        default: hipLaunchKernelGGL((attn_kernel<HT, ROWS_IDX>), grid, dim3(256), 0, s, a); break;
    }
}

// (more than 64 KB of dynamic LDS has to be asked for: 32768 keys per split, caches above 4M rows)
hipError_t prepare_attention(const hata_ctx* c) {
    const void* fn = c->HT == 8   ? (const void*)attn_kernel<8, ROWS_SELECT>
                     : c->HT == 5 ? (const void*)attn_kernel<5, ROWS_SELECT>
                     : c->HT == 4 ? (const void*)attn_kernel<4, ROWS_SELECT>
                     : c->HT == 2 ? (const void*)attn_kernel<2, ROWS_SELECT>
                                  : (const void*)attn_kernel<1, ROWS_SELECT>;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 32768 * 2 + 32);
}

// mode 0: rows from idx (count from k); 2: select on the fly
// from the workspace's scores / thresholds (idx is written)
hipError_t launch_attention(const hata_ctx* c, int mode, const void* q, const void* K,
                            const void* V, int32_t* idx, const int32_t* count_src,
                            const int32_t* seq_len, int B, float sm_scale, void* out,
                            float* out_f32, hipStream_t s) {
    const hata_config& f = c->cfg;
    AttnArgs a;
    a.q = (const uint16_t*)q; a.K = (const uint16_t*)K; a.V = (const uint16_t*)V;
    a.idx_in = idx; a.idx_out = idx; a.count_src = count_src;
    a.scores = c->scores; a.seq_len = seq_len; a.chunk_info = c->chunk_info;
    a.unit_info = c->unit_info; a.chunk = c->chunk; a.n_chunks = c->n_chunks;
    // splits of a selected step: single chunks, paired up while at least 16 splits and 256 workgroups remain (a
    // long cache's many small slices cost more in the merge than they gain; 131072 keys, 8 units, k = 512, 64 / 32 /
    // 16 splits: 29.1 / 25.0 / 26.2 us a step) and to at most 256 splits (n_chunks <= 1024, chunk <= 8192)
    a.chunks_per_split = 1;
    const auto splits = [&](int per) { return (c->n_chunks + per - 1) / per; };
    while (splits(a.chunks_per_split) > 256 ||
           (a.chunks_per_split * c->chunk < 32768 && splits(2 * a.chunks_per_split) >= 16 &&
            (int64_t)splits(2 * a.chunks_per_split) * f.Hkv * (c->G / c->HT) * B >= 256))
        a.chunks_per_split *= 2;
    a.partials = c->partials; a.counter = c->attn_counter; a.counter_stride = c->attn_counter_stride;
    // rows an owner attends over itself: half as many again as it gets of an even spread, in turns of the four waves (64
    // rows); above 512 only where more pieces could not be merged
    a.owners = splits(a.chunks_per_split);
    a.B = B;
    a.piece_rows = 64;
    while ((a.piece_rows < 512 && 2 * (int64_t)a.owners * a.piece_rows < 3 * (int64_t)f.k_max) ||
           a.owners + f.k_max / a.piece_rows > 256 || B + (f.k_max / a.piece_rows * (int64_t)B + a.owners - 1) / a.owners > 65535)
        a.piece_rows += 64;
    const int further = f.k_max / a.piece_rows;
    a.out = (uint16_t*)out; a.out_f32 = out_f32;
    a.Hq = f.Hq; a.Hkv = f.Hkv; a.G = c->G; a.L_cap = f.L_cap; a.k_max = f.k_max;
    a.rows_per_wg = c->sparse_rows;
    a.n_splits = mode == ROWS_SELECT ? a.owners + further : c->sparse_splits;
    a.sb = f.kv_stride_b; a.sh = f.kv_stride_h; a.sn = f.kv_stride_n;
    a.scale_log2 = sm_scale * 1.4426950408889634f;
    const dim3 grid(mode == ROWS_SELECT ? a.owners : a.n_splits, f.Hkv * (c->G / c->HT),
                    mode == ROWS_SELECT ? B + (further * B + a.owners - 1) / a.owners : B);
    switch (c->HT) {
        case 8: launch_mode<8>(mode, a, grid, s); break;
        case 5: launch_mode<5>(mode, a, grid, s); break;
        case 4: launch_mode<4>(mode, a, grid, s); break;
        case 2: launch_mode<2>(mode, a, grid, s); break;
        default: launch_mode<1>(mode, a, grid, s); break;
    }
    return hipGetLastError();
}

}  // namespace hata
