// Decode attention over a list of cache rows (Alg. 3 of the paper: Gather + Attention, with
// the gather fused into the attention kernel; Eq. 2 third line, scale of Eq. 1).
//
// One kernel template, two row sources:
//   ROWS_IDX     rows come from an index list in memory            (hata_sparse_decode)
//   ROWS_SELECT  the rows of one chunk of the cache (a few, of a very long one) that the unit
//                threshold selects: ordered compaction of the chunk's stored scores; its part of
//                the index list is written as a by-product  (hata_decode_step, form without waits)
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
    const int32_t* count_src;   // k[B]
    const uint16_t* scores;     // ROWS_SELECT ...
    const int32_t* seq_len;
    const uint16_t* cum;        // [units, n_chunks, NBP] cumulative histograms of the chunks' scores
    const int32_t* estimate;    // [units, n_chunks] the chunks' estimates of the threshold
    int NBP, chunk, n_chunks, chunks_per_split, owners, piece_rows, B;  // (chunk, chunks_per_split: powers of two)
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
// what the selection needs of a chunk -- its scores, its cumulative histogram -- is at addresses known from
// the start, and on the XCD that scored the chunk.  The unit's threshold and the chunk's place in the index list come from
// 64 columns of all the chunks' cumulative histograms around the chunk's own estimate (as in hata_coop.hip); the scoring launch's
// last workgroup of a unit used to find them, behind everybody else: 2 x 20011 keys, a group of five, 24.6 -> 22.2 us a step
// (the scoring launch 9.8 -> 4.8, this one 10.8 -> 13.8), one sequence of 32768 22.6 -> 20.0, 32 of them 84.4 -> 82.4.  Slices of the index list instead, which had to find their chunks first,
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
    __shared__ uint4 s_win[MODE == ROWS_SELECT ? 4 : 1][64][2];  // {columns 0 and 1 of all chunks, of those before this owner's}, {of this owner's}
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
        const int per = a.chunks_per_split, span = per * a.chunk, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        const uint16_t* hu = a.cum + u * a.n_chunks * a.NBP;
        const bool owner = split < a.owners;
        const int c0 = owner ? split * per : 0;  // the owner's first chunk (a further piece looks from chunk 0)
        const int32_t* estimates = a.estimate + u * a.n_chunks + min(c0, a.n_chunks - 1);
        const int estimate_own = estimates[0], estimate_before = estimates[c0 > 0 && a.n_chunks > 1 ? -1 : 0];
        const int L = clampi(a.seq_len[b], 0, a.L_cap), keff = min(clampi(a.count_src[b], 0, a.k_max), L);
        const int nc = (L + a.chunk - 1) >> __builtin_ctz(a.chunk);
        const int live = (L + span - 1) >> __builtin_ctz(span);      // owners with keys
        int32_t* io = a.idx_out + u * a.k_max;
        if (split == 0) {
            if (ht == 0)  // slots of the index list past the selected count hold -1
                for (int p = keff + tid; p < a.k_max; p += 256) io[p] = -1;
            if (L == 0) zero_output();
        }
        if (owner ? split >= live : live == 0) return;
        const int c1 = min(c0 + per, nc);  // past the owner's last chunk
        auto stage_scores = [&](int base, int n_keys) {
            const uint16_t* sp = a.scores + u * a.L_cap + base;
            const bool whole = (reinterpret_cast<uintptr_t>(sp) & 15) == 0;
            for (int i = tid * 8; i < n_keys; i += 256 * 8) {
                if (whole && i + 8 <= n_keys) {
                    *reinterpret_cast<uint4*>(&s_sc[i]) = *reinterpret_cast<const uint4*>(sp + i);
                } else {
                    for (int e = i; e < min(i + 8, n_keys); ++e) s_sc[e] = sp[e];
                }
            }
        };
        // The threshold T lies in [t_lo, t_hi]; a window of 64 columns shows it if the first of them counts fewer than keff keys (or
        // is score 0) and the last one at least keff.  The next window is beside it, the ones after that halve what is left.
        const int w0_max = max(0, a.NBP - 64);
        // (a last chunk of a few keys knows nothing of the unit: the chunk before does)
        const int estimate = 8 * (L - c0 * a.chunk) < a.chunk ? estimate_before : estimate_own;
        int t_lo = 0, t_hi = a.NBP - 1, w0 = keff == 0 ? 0 : clampi((estimate - 32) & ~1, 0, w0_max);
        int T = 0, need = 0, off = 0, take = 0, cnt = 0;
        bool found = false;
#pragma clang loop unroll(disable)
        for (int it = 0; it < 32 && !found; ++it) {
            // a wave reads two rows at a time, half a wave each, a lane two columns
            const uint16_t* hw = hu + min(w0 + 2 * (lane & 31), a.NBP - 2);
            uint32_t sum[6] = {0, 0, 0, 0, 0, 0};
            constexpr int UN = 8;
            auto request = [&](uint32_t (&x)[UN], int r2) {
#pragma unroll
                for (int j = 0; j < UN; ++j) {
                    x[j] = 0;
                    if (r2 + 8 * j < nc) x[j] = *reinterpret_cast<const uint32_t*>(hw + (int64_t)min(r2 + (lane >> 5) + 8 * j, nc - 1) * a.NBP);
                }
            };
            auto add = [&](const uint32_t (&x)[UN], int r2) {
#pragma unroll
                for (int j = 0; j < UN; ++j) {
                    const int c = r2 + (lane >> 5) + 8 * j;
                    const uint32_t lo = x[j] & 0xffffu, hi = x[j] >> 16;
                    sum[0] += c < nc ? lo : 0u;
                    sum[1] += c < nc ? hi : 0u;
                    sum[2] += c < c0 ? lo : 0u;
                    sum[3] += c < c0 ? hi : 0u;
                    sum[4] += c >= c0 && c < c1 ? lo : 0u;
                    sum[5] += c >= c0 && c < c1 ? hi : 0u;
                }
            };
            for (int r2 = 2 * wv; r2 < nc; r2 += 16 * UN) {  // (the 65th row is no round trip of its own)
                uint32_t x[UN], y[UN];
                request(x, r2);
                const bool more = r2 + 8 * UN < nc;
                if (more) request(y, r2 + 8 * UN);
                add(x, r2);
                if (more) add(y, r2 + 8 * UN);
            }
            if (it == 0 && owner) stage_scores(split * span, min(span, L - split * span));  // (behind the first window's loads)
            if (it) __syncthreads();  // (the last window has been read)
            s_win[wv][lane][0] = make_uint4(sum[0], sum[1], sum[2], sum[3]);
            s_win[wv][lane][1] = make_uint4(sum[4], sum[5], 0, 0);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 6; ++i) sum[i] = 0;
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                const uint4 v = s_win[w >> 1][(w & 1) * 32 + (lane & 31)][0], o = s_win[w >> 1][(w & 1) * 32 + (lane & 31)][1];
                sum[0] += v.x; sum[1] += v.y; sum[2] += v.z; sum[3] += v.w;
                sum[4] += o.x; sum[5] += o.y;
            }
            const unsigned long long hit = __builtin_amdgcn_ballot_w64(sum[1] >= (uint32_t)keff);
            if (hit == 0ull) {
                t_lo = w0 + 64;
            } else {
                const int l = __ffsll(hit) - 1, p = max(l - 1, 0);
                const bool even = (uint32_t)__builtin_amdgcn_readlane((int)sum[0], l) >= (uint32_t)keff;
                if (even && l == 0 && w0 > 0) {
                    t_hi = w0;
                } else {
                    found = true;
                    T = w0 + 2 * l + (even ? 0 : 1);
                    // keys below T and up to T: in the whole unit, in the chunks before the owner's, in the owner's
                    auto below = [&](uint32_t e, uint32_t o) {
                        return even ? (l > 0 ? __builtin_amdgcn_readlane((int)o, p) : 0) : __builtin_amdgcn_readlane((int)e, l);
                    };
                    auto up_to = [&](uint32_t e, uint32_t o) { return __builtin_amdgcn_readlane((int)(even ? e : o), l); };
                    need = keff - below(sum[0], sum[1]);  // ties to grant, in cache order
                    const int lt_b = below(sum[2], sum[3]), eq_b = up_to(sum[2], sum[3]) - lt_b;
                    const int lt = below(sum[4], sum[5]), eq = up_to(sum[4], sum[5]) - lt;
                    take = clampi(need - eq_b, 0, eq);
                    cnt = lt + take;
                    off = lt_b + min(eq_b, need);
                }
            }
            if (!found) w0 = clampi((it == 0 ? (hit ? t_hi - 62 : t_lo - 2) : (t_lo + t_hi) / 2 - 32) & ~1, 0, w0_max);
        }
        // Rows each owner selects, lane l looking at owners l, l + 64, ...: pieces beyond an owner's first; returns how many there
        // are, and finds number `nth` of them: its owner, its place there, and what that owner selects.
        const float half_inv = 0.5f * __builtin_amdgcn_rcpf((float)a.piece_rows);  // (rows - 1) / piece_rows, exact below 2^20
        auto columns = [&](int s, int& lt, int& le) {
            lt = le = 0;
            for (int i = 0; i < per; ++i) {
                const int c = s * per + i;
                if (c < nc) {
                    const uint16_t* row = hu + (int64_t)c * a.NBP;
                    lt += T > 0 ? row[T - 1] : 0;
                    le += row[min(T, a.NBP - 1)];
                }
            }
        };
        int lt0, le0;  // requested here, used behind the attention
        columns(lane, lt0, le0);
        auto further_pieces = [&](int nth, int& own, int& piece, int& off, int& take, int& cnt) {
            int extra = 0, ties = 0, rows_before = 0;  // of the owners before these 64
            for (int s0 = 0; s0 < live; s0 += 64) {
                const int s = s0 + lane;
                int lt = lt0, le = le0;
                if (s0) columns(s, lt, le);
                const int eq = le - lt, eq_incl = (int)wave_incl_scan((uint32_t)eq);
                const int granted = clampi(need - ties - (eq_incl - eq), 0, eq);
                const int rows = keff > 0 ? lt + granted : 0;
                const int more = rows > 0 ? (int)((float)(2 * rows - 1) * half_inv) : 0;
                const int rows_incl = (int)wave_incl_scan((uint32_t)rows);
                const int upto = extra + (int)wave_incl_scan((uint32_t)more);
                const unsigned long long past = __builtin_amdgcn_ballot_w64(upto - more <= nth && upto > nth);
                if (past) {
                    const int l = __ffsll(past) - 1;
                    own = s0 + l;
                    piece = nth - __builtin_amdgcn_readlane(upto - more, l) + 1;
                    off = rows_before + __builtin_amdgcn_readlane(rows_incl - rows, l);
                    take = __builtin_amdgcn_readlane(granted, l);
                    cnt = __builtin_amdgcn_readlane(rows, l);
                }
                extra = __builtin_amdgcn_readlane(upto, 63);
                ties += __builtin_amdgcn_readlane(eq_incl, 63);
                rows_before += __builtin_amdgcn_readlane(rows_incl, 63);
            }
            return min(extra, a.n_splits - a.owners);
        };
        int own = split, piece = 0, extra = 0;
        if (!owner) {
            extra = further_pieces(split - a.owners, own, piece, off, take, cnt);
            if (split - a.owners >= extra) return;
            slot = live + split - a.owners;
        }
        const int base = own * span, n_keys = min(span, L - base);
        off = clampi(off, 0, a.k_max);
        cnt = clampi(cnt, 0, min(n_keys, a.k_max - off));
        if (!owner) stage_scores(base, n_keys);
        __syncthreads();
        if (cnt > 0)  // (the same for the whole workgroup)
            compact_lds(s_sc, n_keys, span / 256, T, take, cnt, scan4, [&](int r, int n) {
                s_sc[r] = (uint16_t)n;
                if (ht == 0 && piece == 0) io[off + r] = base + n;
            });
        __syncthreads();
        attend(piece * a.piece_rows, min(cnt, (piece + 1) * a.piece_rows), [&](int row) { return base + (int)s_sc[row]; });
        if (owner) {
            int o, p, f, t, n;
            extra = further_pieces(-1, o, p, f, t, n);
        }
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
    a.scores = c->scores; a.seq_len = seq_len; a.cum = c->chunk_hist; a.estimate = c->chunk_info; a.NBP = c->NBP;
    a.chunk = c->chunk; a.n_chunks = c->n_chunks;
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
