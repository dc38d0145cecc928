"""The stage kernels at the edges of their launch rules, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hata_oracle as O
from paper_2506_02572_amd import synth
from tests import harness as H


@pytest.mark.parametrize("r,G,max_new", [(32, 1, 1), (64, 3, 8), (96, 5, 2), (128, 16, 3), (256, 16, 7)])
def test_encode_few_vectors(r, G, max_new):
    import torch
    from paper_2506_02572_amd import hata
    B, Hkv, L_cap = 3, 2, 40
    print(f"[stages] encode r={r} G={G} max_new={max_new}", flush=True)
    rng = np.random.default_rng(r + G)
    K = synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L_cap, 128)))
    q = synth.round_to_bf16_bits(rng.standard_normal((B, Hkv * G, 128)))
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    start = np.array([0, L_cap - max_new, 11], np.int32)
    n_new = np.array([max_new, max_new, max_new - 1], np.int32)
    ctx = hata.Context(B, Hkv * G, Hkv, 128, r, L_cap, 8)
    before = rng.integers(0, 2**32, (B, Hkv, L_cap, r // 32), dtype=np.uint32)
    codes = H.to_dev(before.copy())
    ctx.hata_encode_keys(H.to_dev(K), H.to_dev(W), H.to_dev(start), H.to_dev(n_new), B, max_new, codes)
    qcodes = torch.zeros((B, Hkv * G, r // 32), dtype=torch.int32, device="cuda")
    ctx.hata_encode_query(H.to_dev(q), H.to_dev(W), B, qcodes)
    torch.cuda.synchronize()
    ref, near = O.encode_keys_batch(K, W, start, n_new, codes=before.copy())
    H.check_codes(H.to_host(codes, np.uint32), ref, near, "keys")  # (rows outside the range keep their codes)
    H.check_codes(H.to_host(qcodes, np.uint32), *O.encode_query_batch(q, W), "queries")
    ctx.close()


@pytest.mark.parametrize("L_cap", [1, 7, 900, 8192, 8193, 16381, 17003, 32768, 32771, 65533, 65536, 65537])
@pytest.mark.parametrize("kind", ["spread", "ties", "largest"])
def test_selection(L_cap, kind):
    import torch
    from paper_2506_02572_amd import hata
    B, Hkv, G, r = 3, 2, 4, 128
    k_max = max(1, L_cap // 3)
    print(f"[stages] topk L_cap={L_cap} {kind}", flush=True)
    rng = np.random.default_rng(L_cap)
    s = {"spread": rng.normal(256, 12, (B, Hkv, L_cap)), "ties": rng.integers(3, 5, (B, Hkv, L_cap)),
         "largest": rng.integers(508, 513, (B, Hkv, L_cap))}[kind].astype(np.uint16)
    seq = np.array([L_cap, max(0, L_cap - 3), L_cap // 5], np.int32)
    k = np.array([max(1, L_cap // 64), k_max, min(k_max, 40)], np.int32)
    ctx = hata.Context(B, Hkv * G, Hkv, 128, r, L_cap, k_max)
    for offset in (0, 3):  # of the array in its first 16-byte word
        sd = torch.zeros(B * Hkv * L_cap + 8, dtype=torch.int16, device="cuda")[offset:offset + B * Hkv * L_cap]
        sd.copy_(H.to_dev(s).reshape(-1))
        idx = torch.full((B, Hkv, k_max), -7, dtype=torch.int32, device="cuda")
        ctx.hata_topk(sd, H.to_dev(seq), H.to_dev(k), B, idx)
        torch.cuda.synchronize()
        ref = O.topk_batch(s, seq, k, k_max)
        assert np.array_equal(H.to_host(idx), ref)
    ctx.close()


def test_selection_after_a_context_of_fewer_score_values():
    """The LDS a launch may ask for is the kernel's, not a context's: a later, smaller context does not take it away."""
    import torch
    from paper_2506_02572_amd import hata
    k_max = 300
    for L_cap in (32768, 65536):
        print(f"[stages] two contexts, L_cap={L_cap}", flush=True)
        first = hata.Context(1, 16, 1, 128, 256, L_cap, k_max)
        later = hata.Context(1, 1, 1, 128, 32, L_cap, k_max)
        rng = np.random.default_rng(L_cap)
        seq, k = np.array([L_cap], np.int32), np.array([k_max], np.int32)
        for ctx, top in ((later, 33), (first, 4097)):
            s = rng.integers(top // 2, top, (1, 1, L_cap)).astype(np.uint16)
            idx = torch.full((1, 1, k_max), -7, dtype=torch.int32, device="cuda")
            ctx.hata_topk(H.to_dev(s), H.to_dev(seq), H.to_dev(k), 1, idx)
            torch.cuda.synchronize()
            assert np.array_equal(H.to_host(idx), O.topk_batch(s, seq, k, k_max))
            ctx.close()


@pytest.mark.parametrize("L,k_max,chunk", [(1, 1, 0), (1024, 200, 1024), (1025, 1025, 1024), (20011, 700, 1024),
                                           (40000, 512, 1024), (40000, 3000, 8192)])
@pytest.mark.parametrize("heads", [(5, 1), (2, 2), (8, 1)])
def test_chunk_owned_attention(L, k_max, chunk, heads):
    Hq, Hkv = heads
    B = 2
    w = synth.Workload("chunks", B, Hq, Hkv, 128, 64, (L, max(1, L // 3)), (k_max, max(1, k_max // 2)), k_max=k_max)
    print(f"[stages] attention L={L} k={k_max} chunk={chunk} heads={heads}", flush=True)
    c = H.Case(w, shared_device=True, chunk=chunk)
    c.ctx.hata_set_step_mode(3)
    assert c.ctx.hata_step_plan(B)[0] == 3
    q = c.inp.q()
    for clustered in (False, True):
        codes = c.codes_ref.copy()
        if clustered:  # half of the budget's rows in one run are as near as can be: one chunk or two hold them all
            qc, _ = O.encode_query_batch(q, c.inp.W_H)
            codes[:, :, L // 2: L // 2 + k_max // 2] = qc.reshape(B, Hkv, Hq // Hkv, -1)[:, :, :1]
        cd = H.to_dev(codes.copy())
        out, out32 = c.empty((B, Hq, 128), c.torch.int16), c.empty((B, Hq, 128), c.torch.float32)
        c.ctx.hata_decode_step(H.to_dev(q), c.K, c.V, c.W_H, cd, c.seq_len, c.k, B, True, c.scale, out, out32)
        c.sync()
        ref = O.decode_step(q, c.inp.K, c.inp.V, c.inp.W_H, codes, c.inp.seq_len, c.inp.k, k_max, c.scale, append=True)
        assert np.array_equal(H.to_host(cd, np.uint32), codes)
        assert np.array_equal(H.to_host(c.ctx.hata_step_buffers()[2]), ref["idx"])
        H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), ref["out"], "step")
    c.ctx.close()


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8, 16])
@pytest.mark.parametrize("lens", [(1, 0, 15), (16, 17, 127), (129, 128, 2047), (4099, 20000, 300)])
def test_dense_attention(G, lens):
    import torch
    from paper_2506_02572_amd import hata
    B, Hkv, L_cap = len(lens), 2, max(lens)
    print(f"[stages] dense G={G} lens={lens}", flush=True)
    rng = np.random.default_rng(G)
    # rows of the caches interleaved over the KV heads: [B, L_cap, Hkv, 128]
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, L_cap, Hkv, 128))) for _ in range(2))
    q = synth.round_to_bf16_bits(rng.standard_normal((B, Hkv * G, 128)) * 3)
    seq = np.array(lens, np.int32)
    ctx = hata.Context(B, Hkv * G, Hkv, 128, 64, L_cap, 1, kv_strides=(L_cap * Hkv * 128, 128, Hkv * 128))
    out = torch.full((B, Hkv * G, 128), -7, dtype=torch.int16, device="cuda")
    out32 = torch.full((B, Hkv * G, 128), 7.0, dtype=torch.float32, device="cuda")
    for _ in range(2):  # (the second call finds the arrival counters as the first one left them)
        ctx.hata_dense_decode(H.to_dev(q), H.to_dev(K), H.to_dev(V), H.to_dev(seq), B, 128 ** -0.5, out, out32)
    torch.cuda.synchronize()
    ref = O.dense_decode_batch(q, K.transpose(0, 2, 1, 3), V.transpose(0, 2, 1, 3), seq, 128 ** -0.5)
    H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), np.where(seq[:, None, None] > 0, ref, 0.0), "dense")
    ctx.close()


@pytest.mark.parametrize("r", [32, 64, 128, 256])
@pytest.mark.parametrize("max_new", [9, 63, 64, 65, 129, 300, 1025])
def test_fill_and_encode_many_keys(r, max_new):
    """Remainders of a stage and of a workgroup's keys; with prepared weights and without, both layouts."""
    import torch
    from paper_2506_02572_amd import hata
    B, Hkv, P, first = 3, 2, 16, 5
    L_cap = -(-(max_new + first) // P) * P
    blocks = L_cap // P
    rng = np.random.default_rng(r + max_new)
    K_new, V_new = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, max_new, 128))) for _ in range(2))
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    start = np.array([0, first, L_cap - max_new // 2], np.int32)  # (the last one does not fit whole)
    n_new = np.array([max_new, max_new - 1, max_new], np.int32)
    K0, V0 = (rng.integers(0, 2**16, (B, Hkv, L_cap, 128), dtype=np.uint16) for _ in range(2))
    K_ref, V_ref = K0.copy(), V0.copy()
    for b in range(B):
        n = min(int(n_new[b]), L_cap - int(start[b]))
        K_ref[b, :, start[b]:start[b] + n], V_ref[b, :, start[b]:start[b] + n] = K_new[b, :, :n], V_new[b, :, :n]
    before = rng.integers(0, 2**32, (B, Hkv, L_cap, r // 32), dtype=np.uint32)
    n_fit = np.minimum(n_new, L_cap - start).astype(np.int32)
    ref, near = O.encode_keys_batch(K_ref, W, start, n_fit, codes=before.copy())
    pages = rng.permutation(B * blocks).astype(np.int32).reshape(B, blocks)
    Wd, st, nn = H.to_dev(W), H.to_dev(start), H.to_dev(n_new)

    def pool(a):  # [B, Hkv, L_cap, x] -> pages [B * blocks, Hkv, P, x]
        out = np.empty((B * blocks, Hkv, P, a.shape[-1]), a.dtype)
        out[pages.reshape(-1)] = a.reshape(B, Hkv, blocks, P, -1).transpose(0, 2, 1, 3, 4).reshape(B * blocks, Hkv, P, -1)
        return out

    ctx = hata.Context(B, 2 * Hkv, Hkv, 128, r, L_cap, 8)
    for prepared in (False, True):
        print(f"[stages] fill r={r} max_new={max_new} prepared={prepared}", flush=True)
        if prepared:
            ctx.hata_prepare_weights(Wd)
        codes = H.to_dev(before.copy())
        ctx.hata_encode_keys(H.to_dev(K_ref), Wd, st, nn, B, max_new, codes)
        H.check_codes(H.to_host(codes, np.uint32), ref, near, "keys in the cache")
        K, V, codes = H.to_dev(K0.copy()), H.to_dev(V0.copy()), H.to_dev(before.copy())
        ctx.hata_prefill_write(H.to_dev(K_new), H.to_dev(V_new), st, nn, B, max_new, K, V, codes, Wd)
        H.check_codes(H.to_host(codes, np.uint32), ref, near, "fill")
        assert np.array_equal(H.to_host(K, np.uint16), K_ref) and np.array_equal(H.to_host(V, np.uint16), V_ref)
        K, V, codes = H.to_dev(pool(K0)), H.to_dev(pool(V0)), H.to_dev(pool(before))
        ctx.hata_prefill_write_paged(H.to_dev(K_new), H.to_dev(V_new), st, nn, B, max_new, K, V, codes,
                                     H.to_dev(pages), blocks, P, B * blocks, Wd)
        assert np.array_equal(H.to_host(K, np.uint16), pool(K_ref)) and np.array_equal(H.to_host(V, np.uint16), pool(V_ref))
        H.check_codes(H.to_host(codes, np.uint32), pool(ref), pool(near), "paged fill")
    ctx.close()


@pytest.mark.parametrize("r", [32, 64, 128, 256])
def test_encode_keys_of_many_units(r):
    """Workgroups of many keys (512 units), ranges of all lengths round the 128 keys of a stage."""
    import torch
    from paper_2506_02572_amd import hata
    B, Hkv, max_new, L_cap = 64, 8, 270, 280
    print(f"[stages] encode r={r}, 512 units", flush=True)
    rng = np.random.default_rng(r)
    K = synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L_cap, 128), dtype=np.float32))
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    start = rng.integers(0, L_cap - max_new + 1, B).astype(np.int32)
    n_new = np.concatenate([[0, 1, 63, 64, 65, 127, 128, 129, 255, 256, 257, max_new], rng.integers(1, max_new, B - 12)]).astype(np.int32)
    before = rng.integers(0, 2**32, (B, Hkv, L_cap, r // 32), dtype=np.uint32)
    ctx = hata.Context(B, 2 * Hkv, Hkv, 128, r, L_cap, 8)
    Wd = H.to_dev(W)
    ctx.hata_prepare_weights(Wd)
    codes = H.to_dev(before.copy())
    ctx.hata_encode_keys(H.to_dev(K), Wd, H.to_dev(start), H.to_dev(n_new), B, max_new, codes)
    torch.cuda.synchronize()
    ref, near = O.encode_keys_batch(K, W, start, n_new, codes=before.copy(), bulk=True)
    H.check_codes(H.to_host(codes, np.uint32), ref, near, "keys")
    ctx.close()


# groups whose weights stay fp32: no tile of four heads or more divides them
FP32_GROUPS = [1, 2, 3, 6, 7, 9, 11, 13, 14]


def dense(G, q, K, V, seq):
    """One KV head per sequence; q, K, V as fp32 arrays of bf16 values.  Returns the fp32 and the bf16 output."""
    import torch
    from paper_2506_02572_amd import hata
    B, L_cap = K.shape[0], K.shape[1]
    ctx = hata.Context(B, G, 1, 128, 64, L_cap, 1)
    out = torch.full((B, G, 128), -7, dtype=torch.int16, device="cuda")
    out32 = torch.full((B, G, 128), 7.0, dtype=torch.float32, device="cuda")
    qd, Kd, Vd = (H.to_dev(synth.round_to_bf16_bits(x)) for x in (q, K, V))
    ctx.hata_dense_decode(qd, Kd, Vd, H.to_dev(seq), B, 128 ** -0.5, out, out32)
    torch.cuda.synchronize()
    ctx.close()
    return H.to_host(out32), H.to_host(out, np.uint16)


@pytest.mark.parametrize("G", FP32_GROUPS)
def test_dense_weights_are_fp32(G):
    """All values 1: the output is sum(w) / sum(w), 1 up to the rounding of the two sums.  Up to 41 rows a wave adds at
    most 16 products per channel or 4 weights per lane and 4 lanes, then 8 waves and slices are merged: fewer than 40
    roundings of 2^-24 in all, 2.4e-6.  Weights cut to 16 bits would be short by 5e-6 on average."""
    print(f"[stages] dense weights G={G}", flush=True)
    rng = np.random.default_rng(G)
    seq = np.array([5, 16, 41, 33], np.int32)
    K = rng.standard_normal((len(seq), 41, 128)).astype(np.float32)
    q = (0.1 * rng.standard_normal((len(seq), G, 128))).astype(np.float32)
    out32, out = dense(G, q, K, np.ones_like(K), seq)
    assert np.max(np.abs(out32.astype(np.float64) - 1.0)) <= 40 * 2.0 ** -24
    assert np.all(out == 0x3f80)


@pytest.mark.parametrize("G", FP32_GROUPS)
@pytest.mark.parametrize("L", [3, 40, 700])
def test_dense_with_infinite_values(G, L):
    """Infinite values in rows that count, the one with the largest score (weight exactly 1) among them: infinite outputs
    of their sign in those channels, nothing elsewhere.  Rows past the end are infinite too, and do not count."""
    print(f"[stages] dense infinities G={G} L={L}", flush=True)
    rng = np.random.default_rng(L + G)
    K = rng.standard_normal((1, L + 20, 128)).astype(np.float32)
    q = (0.3 * rng.standard_normal((1, G, 128))).astype(np.float32)
    V = rng.standard_normal(K.shape).astype(np.float32)
    V[:, L:] = np.inf
    finite = V[0].copy()
    bits = synth.round_to_bf16_bits(q), synth.round_to_bf16_bits(K)
    qf, Kf = (synth.bf16_to_f32(b).astype(np.float64) for b in bits)
    best = int(np.argmax(Kf[0, :L] @ qf[0, 0]))  # of the first head
    V[0, best, 5], V[0, best, 127], V[0, (best + 1) % L, 64] = np.inf, -np.inf, np.inf
    out32, _ = dense(G, q, K, V, np.array([L], np.int32))
    assert np.all(out32[0, :, [5, 64]] == np.inf) and np.all(out32[0, :, 127] == -np.inf)
    s = qf[0] @ Kf[0, :L].T * 128 ** -0.5
    w = np.exp(s - s.max(1, keepdims=True))
    ref = w @ synth.bf16_to_f32(synth.round_to_bf16_bits(finite[:L])).astype(np.float64) / w.sum(1, keepdims=True)
    rest = np.setdiff1d(np.arange(128), [5, 64, 127])
    assert np.max(np.abs(out32[0][:, rest] - ref[:, rest])) <= H.ABS_TOL


def shortest_us(call, turns=9, per_turn=5):
    import torch
    call()
    times = []
    for _ in range(turns):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(per_turn):
            call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1000 / per_turn)
    return min(times)


@pytest.mark.parametrize("B,Hkv,G", [(2, 1, 4), (2, 8, 1), (64, 1, 5), (65, 3, 2), (130, 5, 1), (200, 1, 3)])
@pytest.mark.parametrize("lens", ["one_long", "spread", "equal", "empty"])
def test_dense_shares_of_unequal_sequences(B, Hkv, G, lens):
    """Batches on both sides of the 64 sequences a wave looks at together, and of one workgroup per unit."""
    import torch
    from paper_2506_02572_amd import hata
    L_cap = 2500 if B * Hkv < 64 else 900
    print(f"[stages] dense shares B={B} Hkv={Hkv} {lens}", flush=True)
    rng = np.random.default_rng(B + G)
    seq = {"one_long": np.where(np.arange(B) == B // 2, L_cap, rng.integers(0, 40, B)), "spread": rng.integers(0, L_cap + 1, B),
           "equal": np.full(B, 333), "empty": np.where(np.arange(B) == B - 1, 129, 0)}[lens].astype(np.int32)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L_cap, 128), dtype=np.float32)) for _ in range(2))
    q = synth.round_to_bf16_bits(rng.standard_normal((B, Hkv * G, 128)) * 2)
    ctx = hata.Context(B, Hkv * G, Hkv, 128, 32, L_cap, 1)
    out = torch.full((B, Hkv * G, 128), -7, dtype=torch.int16, device="cuda")
    out32 = torch.full((B, Hkv * G, 128), 7.0, dtype=torch.float32, device="cuda")
    qd, Kd, Vd, sd = (H.to_dev(x) for x in (q, K, V, seq))
    for _ in range(2):
        ctx.hata_dense_decode(qd, Kd, Vd, sd, B, 128 ** -0.5, out, out32)
    torch.cuda.synchronize()
    ref = O.dense_decode_batch(q, K, V, seq, 128 ** -0.5)
    H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), np.where(seq[:, None, None] > 0, ref, 0.0), "dense")
    ctx.close()


def test_dense_spreads_the_one_long_sequence_of_a_batch():
    """One sequence of 32768 rows among 15 of 512 costs about what it costs alone (1.35 times); cut by what the other sequences
    could hold instead of what they hold, its stream runs on a sixteenth of the chip (5.8 times)."""
    import torch
    from paper_2506_02572_amd import hata
    B, Hkv, G, L = 16, 8, 4, 32768
    K, V = (torch.randn((B, Hkv, L, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    q = torch.randn((B, Hkv * G, 128), dtype=torch.bfloat16, device="cuda")
    out = torch.zeros_like(q)
    seq = torch.full((B,), 512, dtype=torch.int32, device="cuda")
    seq[0] = L
    alone, batch = hata.Context(1, Hkv * G, Hkv, 128, 32, L, 1), hata.Context(B, Hkv * G, Hkv, 128, 32, L, 1)
    t_alone = shortest_us(lambda: alone.hata_dense_decode(q, K, V, seq, 1, 128 ** -0.5, out))
    t_batch = shortest_us(lambda: batch.hata_dense_decode(q, K, V, seq, B, 128 ** -0.5, out))
    print(f"[stages] dense alone {t_alone:.1f} us, in the batch {t_batch:.1f} us", flush=True)
    assert t_batch < 3 * t_alone
    alone.close()
    batch.close()


@pytest.mark.parametrize("L,k_max,chunk", [(2100, 2100, 0), (3000, 1000, 0), (9000, 4000, 1024), (30000, 600, 8192), (70000, 700, 1024)])
@pytest.mark.parametrize("heads", [(5, 1), (2, 2), (8, 1), (4, 4)])
def test_selected_rows_of_one_chunk_in_pieces(L, k_max, chunk, heads):
    """Runs of selected rows that fill a chunk and more, so that the chunk's rows go to several workgroups."""
    Hq, Hkv = heads
    B = 3
    w = synth.Workload("pieces", B, Hq, Hkv, 128, 64, (L, max(1, L // 3), 5), (k_max, max(1, k_max // 2), 3), k_max=k_max)
    print(f"[stages] pieces L={L} k={k_max} chunk={chunk} heads={heads}", flush=True)
    c = H.Case(w, shared_device=True, chunk=chunk)
    c.ctx.hata_set_step_mode(3)
    assert c.ctx.hata_step_plan(B)[0] == 3
    q = c.inp.q()
    qc, _ = O.encode_query_batch(q, c.inp.W_H)
    near = qc.reshape(B, Hkv, Hq // Hkv, -1)[:, :, :1]
    for first, count in ((0, k_max), (L // 4, k_max), (L // 4 - 700, k_max // 2 + 1), (L // 3 - 65, 65), (L // 3 - 200, 129)):
        codes = c.codes_ref.copy()
        codes[:, :, max(0, first): max(0, first) + count] = near
        cd = H.to_dev(codes.copy())
        out, out32 = c.empty((B, Hq, 128), c.torch.int16), c.empty((B, Hq, 128), c.torch.float32)
        for _ in range(2):  # (the second call finds the arrival counters as the first one left them)
            c.ctx.hata_decode_step(H.to_dev(q), c.K, c.V, c.W_H, cd, c.seq_len, c.k, B, False, c.scale, out, out32)
        c.sync()
        ref = O.decode_step(q, c.inp.K, c.inp.V, c.inp.W_H, codes, c.inp.seq_len, c.inp.k, k_max, c.scale, append=False)
        assert np.array_equal(H.to_host(c.ctx.hata_step_buffers()[2]), ref["idx"])
        H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), ref["out"], "step")
    c.ctx.close()


def test_selected_rows_in_one_place_are_no_serial_work():
    """2048 selected rows in a row of a 131072-key cache: 1.1 times the step with the rows spread out (2.1 times when one
    workgroup attends over all rows of a chunk)."""
    import torch
    from paper_2506_02572_amd import hata
    Hq, Hkv, L, k, r = 32, 8, 131072, 2048, 256
    K, V = (torch.randn((1, Hkv, L, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    q = torch.randn((1, Hq, 128), dtype=torch.bfloat16, device="cuda")
    W = torch.randn((Hkv, 128, r), device="cuda")
    ctx = hata.Context(1, Hq, Hkv, 128, r, L, k, shared_device=True)
    seq, budget, zero = (torch.tensor([x], dtype=torch.int32, device="cuda") for x in (L, k, 0))
    codes = torch.zeros((1, Hkv, L, r // 32), dtype=torch.int32, device="cuda")
    qcodes = torch.zeros((1, Hq, r // 32), dtype=torch.int32, device="cuda")
    out = torch.zeros_like(q)
    ctx.hata_encode_keys(K, W, zero, seq, 1, L, codes)
    ctx.hata_encode_query(q, W, 1, qcodes)

    def step():
        ctx.hata_decode_step(q, K, V, W, codes, seq, budget, 1, False, 128 ** -0.5, out)

    t_spread = shortest_us(step)
    codes[:, :, L // 2:L // 2 + k] = qcodes.view(1, Hkv, Hq // Hkv, -1)[:, :, :1]
    t_run = shortest_us(step)
    print(f"[stages] rows spread {t_spread:.1f} us, in one place {t_run:.1f} us", flush=True)
    assert t_run < 1.5 * t_spread
    ctx.close()


@pytest.mark.parametrize("r", [32, 64, 128, 256])
def test_codes_of_keys_with_nan(r):
    """A projection that is no number is not >= 0: all code bits 0, whatever the NaN's sign and whichever kernel encodes."""
    import torch
    from paper_2506_02572_amd import hata
    L = 300
    print(f"[stages] NaN keys r={r}", flush=True)
    K = torch.randn((1, 2, L, 128), device="cuda").to(torch.bfloat16)
    K[:, :, 7, 3], K[:, :, 200, 100] = float("nan"), -float("nan")
    W = torch.randn((2, 128, r), device="cuda")
    ctx = hata.Context(1, 4, 2, 128, r, L, 8)
    start, n = (torch.tensor([x], dtype=torch.int32, device="cuda") for x in (0, L))
    for prepared in (False, True):
        if prepared:
            ctx.hata_prepare_weights(W)
        bulk, fill = (torch.full((1, 2, L, r // 32), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        ctx.hata_encode_keys(K, W, start, n, 1, L, bulk)
        ctx.hata_prefill_write(K, K, start, n, 1, L, torch.zeros_like(K), torch.zeros_like(K), fill, W)
        for codes in (bulk, fill):
            assert not codes[:, :, [7, 200]].any() and codes[:, :, 8].any()
    for row in (7, 200):
        one = torch.full((1, 2, L, r // 32), -1, dtype=torch.int32, device="cuda")
        ctx.hata_encode_keys(K, W, start + row, n * 0 + 1, 1, 1, one)
        assert not one[:, :, row].any()
    ctx.close()
