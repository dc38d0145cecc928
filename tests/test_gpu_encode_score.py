"""The launch of a shared device's step that encodes and scores: one, two and four chunks a workgroup, and batches beyond it, against the
stage calls -- query codes, the appended key's code, every score and the selection are the same words."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


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
