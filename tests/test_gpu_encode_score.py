"""The launch of a shared device's step that encodes and scores: one, two and four chunks a workgroup, and batches beyond it, against the
stage calls -- query codes, the appended key's code, every score and the selection are the same words -- and against the oracle, with
caches of any strides and the attention behind it."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hata_oracle as O
from paper_2506_02572_amd import synth
from tests import harness as H


def chunks_of_a_workgroup(ctx, B, Hq, Hkv, r):
    """The rule of the launch (launch_encode_score): 1, 2 or 4 chunks, 0 where encoding has a launch of its own."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    launches, _, n_chunks = ctx.hata_step_plan(B)
    assert launches == 3
    if r not in (32, 64, 128) or Hq // Hkv not in (1, 2, 4, 5, 8):
        return 0
    return next((c for c in (1, 2, 4) if -(-n_chunks // c) * Hkv * B <= cus), 0)


@pytest.mark.parametrize("B,Hq,Hkv,r,L_cap,chunks", [
    (1, 8, 8, 32, 17000, 1), (2, 4, 2, 64, 16500, 1), (3, 8, 2, 128, 20011, 1), (2, 10, 2, 128, 17409, 1), (3, 16, 2, 128, 16390, 1),
    (4, 32, 8, 128, 17000, 2), (4, 40, 8, 64, 17000, 2), (4, 8, 8, 32, 17000, 2),
    (16, 32, 8, 128, 17000, 4), (16, 8, 8, 64, 17000, 4), (16, 64, 8, 128, 17000, 4),
    (4, 32, 8, 256, 17000, 0), (1, 8, 2, 256, 20011, 0), (32, 16, 8, 128, 17000, 0), (2, 6, 2, 128, 20011, 0)])
def test_which_launch_takes_these_shapes(B, Hq, Hkv, r, L_cap, chunks):
    """Those of the test below, on 256 compute units, and a group of three."""
    from paper_2506_02572_amd import hata
    ctx = hata.Context(B, Hq, Hkv, 128, r, L_cap, 200, shared_device=True)
    assert chunks_of_a_workgroup(ctx, B, Hq, Hkv, r) == chunks
    ctx.close()


@pytest.mark.parametrize("append", [True, False])
@pytest.mark.parametrize("B,G,Hkv,r,L_cap,chunks", [
    (3, 1, 2, 32, 5003, 1), (3, 2, 2, 64, 5003, 1), (3, 4, 2, 128, 5003, 1), (3, 5, 2, 128, 5003, 1), (3, 8, 2, 64, 5003, 1), (3, 4, 2, 256, 5003, 0),
    (2, 4, 8, 64, 17409, 2), (2, 5, 8, 32, 17409, 2), (4, 8, 8, 128, 17409, 4), (4, 1, 8, 64, 17409, 4)])
def test_padded_caches_against_the_oracle(B, G, Hkv, r, L_cap, chunks, append):
    """Heads beside each other in a row of 136 and more values, with NaN behind each head's 128: codes, scores, selection and output."""
    import torch
    from paper_2506_02572_amd import hata
    print(f"[encode_score] strided B={B} G={G} Hkv={Hkv} r={r} L_cap={L_cap} append={append}", flush=True)
    k_max, scale, rng = 150, 1.0 / math.sqrt(128), np.random.default_rng(r + G + L_cap)
    pitch, sb = 136, L_cap * Hkv * 136 + 72
    seq = np.array([L_cap, 1025, 1, 4096][:B], np.int32)
    kb = np.array([k_max, 70, 5, k_max][:B], np.int32)
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    q = synth.round_to_bf16_bits(rng.standard_normal((B, Hkv * G, 128)).astype(np.float32))
    codes = rng.integers(0, 2**32, (B, Hkv, L_cap, r // 32), dtype=np.uint32)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L_cap, 128), dtype=np.float32)) for _ in range(2))
    padded = []
    for x in (K, V):
        p = np.full((B, sb), 0x7FC0, np.uint16)
        p[:, :L_cap * Hkv * pitch].reshape(B, L_cap, Hkv, pitch)[..., :128] = x.transpose(0, 2, 1, 3)
        padded.append(H.to_dev(p))
    ref_codes = codes.copy()
    ref = O.decode_step(q, K, V, W, ref_codes, seq, kb, k_max, scale, append=append)
    ctx = hata.Context(B, Hkv * G, Hkv, 128, r, L_cap, k_max, kv_strides=(sb, pitch, Hkv * pitch), shared_device=True, chunk=1024)
    ctx.hata_set_step_mode(3)
    assert chunks_of_a_workgroup(ctx, B, Hkv * G, Hkv, r) == chunks
    cd = H.to_dev(codes)
    out, out32 = (torch.empty((B, Hkv * G, 128), dtype=t, device="cuda") for t in (torch.int16, torch.float32))
    ctx.hata_decode_step(H.to_dev(q), *padded, H.to_dev(W), cd, H.to_dev(seq), H.to_dev(kb), B, append, scale, out, out32)
    torch.cuda.synchronize()
    qcodes, scores, idx = ctx.hata_step_buffers()
    assert np.array_equal(H.to_host(cd, np.uint32), ref_codes)
    assert np.array_equal(H.to_host(qcodes, np.uint32).reshape(ref["qcodes"].shape), ref["qcodes"])
    scores = H.to_host(scores, np.uint16).reshape(ref["scores"].shape)
    for b in range(B):
        assert np.array_equal(scores[b, :, :seq[b]], ref["scores"][b, :, :seq[b]]), b
    assert np.array_equal(H.to_host(idx).reshape(ref["idx"].shape), ref["idx"])
    H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), ref["out"], "strided")
    ctx.close()


@pytest.mark.parametrize("append", [True, False])
@pytest.mark.parametrize("B,Hq,Hkv,r,L_cap", [
    (1, 8, 8, 32, 17000), (2, 4, 2, 64, 16500), (3, 8, 2, 128, 20011), (2, 10, 2, 128, 17409), (3, 16, 2, 128, 16390),  # one chunk a workgroup
    (4, 32, 8, 128, 17000), (4, 40, 8, 64, 17000), (4, 8, 8, 32, 17000),                                         # two
    (16, 32, 8, 128, 17000), (16, 8, 8, 64, 17000), (16, 64, 8, 128, 17000),                                     # four
    (4, 32, 8, 256, 17000), (1, 8, 2, 256, 20011), (32, 16, 8, 128, 17000)])                                   # two launches
def test_encode_and_score_in_one_launch(B, Hq, Hkv, r, L_cap, append):
    import torch
    from paper_2506_02572_amd import hata
    print(f"[encode_score] B={B} Hq={Hq} Hkv={Hkv} r={r} L_cap={L_cap} append={append}", flush=True)
    k_max, scale = 200, 1.0 / math.sqrt(128)
    g = torch.Generator(device="cuda").manual_seed(B * 1000 + Hq + r)
    K = torch.randn((B, Hkv, L_cap, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    V = torch.randn((B, Hkv, L_cap, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    q = torch.randn((B, Hq, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    W = torch.randn((Hkv, 128, r), dtype=torch.float32, device="cuda", generator=g)
    # lengths on both sides of chunks of 1024, 2048 and 4096 keys, an empty sequence, a full one
    some = [L_cap, 4097, 0, 8192, 1, 8193, 2048, 1025, 16384, 4096, 12289, 1024]
    lens = np.array([some[(i * 5) % len(some)] if i else L_cap for i in range(B)], np.int32)
    seq = torch.from_numpy(lens).cuda()
    kb = torch.from_numpy(np.minimum(lens, [k_max - i for i in range(B)]).astype(np.int32)).cuda()
    rows = seq - 1 if append else seq  # coded before the step
    zero = torch.zeros(B, dtype=torch.int32, device="cuda")
    ctx = hata.Context(B, Hq, Hkv, 128, r, L_cap, k_max, shared_device=True)
    codes = torch.zeros((B, Hkv, L_cap, r // 32), dtype=torch.int32, device="cuda")
    ctx.hata_encode_keys(K, W, zero, torch.clamp(rows, min=0), B, L_cap, codes)
    want_codes = codes.clone()
    if append:  # the appended rows by the call for single rows
        live = torch.clamp(seq, max=1)
        ctx.hata_encode_keys(K, W, torch.clamp(seq - 1, min=0), live, B, 1, want_codes)
    out = torch.empty((B, Hq, 128), dtype=torch.bfloat16, device="cuda")
    for _ in range(2):
        ctx.hata_decode_step(q, K, V, W, codes, seq, kb, B, append, scale, out)
    torch.cuda.synchronize()
    assert ctx.hata_step_plan(B)[0] == 3
    qcodes, scores, idx = (t.clone() for t in ctx.hata_step_buffers())
    want_q = torch.zeros_like(qcodes)
    want_s, want_i = torch.zeros_like(scores), torch.zeros_like(idx)
    ctx.hata_encode_query(q, W, B, want_q)
    ctx.hata_hamming_score(want_q, want_codes, seq, B, want_s)
    ctx.hata_topk(want_s, seq, kb, B, want_i)
    torch.cuda.synchronize()
    assert torch.equal(codes, want_codes)
    assert torch.equal(qcodes.view(want_q.shape), want_q)
    scores = scores.view(want_s.shape)
    for b in range(B):
        assert torch.equal(scores[b, :, :lens[b]], want_s[b, :, :lens[b]]), b
    assert torch.equal(idx.view(want_i.shape), want_i)
    ctx.close()


@pytest.mark.parametrize("L_cap,G,r", [(17000, 4, 128), (16500, 1, 32), (20011, 5, 64), (20011, 4, 256)])
def test_sequence_longer_than_its_cache_appends_nothing(L_cap, G, r):
    """The appended row would lie past the cache: no code is written, and the rows that are there are scored with the codes they have."""
    import torch
    from paper_2506_02572_amd import hata
    print(f"[encode_score] L_cap={L_cap} G={G} r={r}, lengths beyond it", flush=True)
    B, Hkv, k_max = 2, 2, 64
    g = torch.Generator(device="cuda").manual_seed(L_cap + r)
    K, V = (torch.randn((B, Hkv, L_cap, 128), dtype=torch.bfloat16, device="cuda", generator=g) for _ in range(2))
    q = torch.randn((B, Hkv * G, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    W = torch.randn((Hkv, 128, r), dtype=torch.float32, device="cuda", generator=g)
    codes = torch.randint(-2**31, 2**31 - 1, (B, Hkv, L_cap, r // 32), dtype=torch.int32, device="cuda", generator=g)
    seq = torch.tensor([L_cap + 1, L_cap + 500], dtype=torch.int32, device="cuda")
    kb = torch.full((B,), k_max, dtype=torch.int32, device="cuda")
    ctx = hata.Context(B, Hkv * G, Hkv, 128, r, L_cap, k_max, shared_device=True)
    want = codes.clone()
    out = torch.empty((B, Hkv * G, 128), dtype=torch.bfloat16, device="cuda")
    ctx.hata_decode_step(q, K, V, W, codes, seq, kb, B, True, 1.0 / math.sqrt(128), out)
    torch.cuda.synchronize()
    assert torch.equal(codes, want)
    qcodes, scores, idx = ctx.hata_step_buffers()
    want_s, want_i = torch.zeros_like(scores).view(B, Hkv, L_cap), torch.zeros_like(idx).view(B, Hkv, k_max)
    ctx.hata_hamming_score(qcodes.clone(), want, seq, B, want_s)
    ctx.hata_topk(want_s, seq, kb, B, want_i)
    torch.cuda.synchronize()
    assert torch.equal(scores.view(want_s.shape), want_s) and torch.equal(idx.view(want_i.shape), want_i)
    ctx.close()
