"""The launch that encodes and scores, with its workgroups dealt out by the sequences' lengths where the cache's size gives them four chunks: one,
two or four in the same grid, against the stage calls -- codes, every score and the selection are the same words."""
import math

import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_encode_score import chunks_of_a_workgroup


def chunks_by_length(n_chunks, chunk, most, lens):
    """The rule (place_by_length): the fewest chunks a workgroup with which the lengths' workgroups fit the grid that the cache's size gives."""
    if most < 4:
        return most
    slots = -(-n_chunks // most) * len(lens)
    return next(c for c in (1, 2, 4) if c == most or sum(max(1, -(-(-(-n // chunk)) // c)) for n in lens) <= slots)


def batch(kind, B, L_cap):
    short = [500, 0, 1, 4096, 4097, 900]
    if kind == "one": return [short[b % 6] for b in range(B - 1)] + [L_cap]
    if kind == "first": return [L_cap] + [500] * (B - 1)
    if kind == "half": return [L_cap if b % 2 else 1000 for b in range(B)]
    if kind == "most": return [L_cap if b % 8 else 700 for b in range(B)]
    if kind == "beyond": return [L_cap + 300 if b % 5 == 2 else short[b % 6] for b in range(B)]  # longer than the cache: nothing is appended
    return [L_cap] * B


@pytest.mark.parametrize("append", [True, False])
@pytest.mark.parametrize("B,Hq,Hkv,r,L_cap,kind,chunks", [
    (4, 32, 8, 128, 17000, "one", 2), (70, 2, 1, 64, 17000, "half", 2),                                                      # two by the cache's size
    (16, 32, 8, 128, 17000, "one", 1), (16, 64, 8, 128, 17000, "first", 1), (16, 32, 8, 64, 17000, "half", 2),               # four
    (16, 40, 8, 128, 17000, "most", 4), (16, 8, 8, 128, 17000, "beyond", 1), (12, 16, 8, 32, 17000, "all", 4),
    (90, 2, 1, 64, 17000, "one", 1), (128, 1, 1, 128, 17000, "most", 4), (100, 1, 1, 32, 17000, "beyond", 1), (100, 1, 1, 32, 17000, "half", 2), (100, 1, 1, 32, 17000, "most", 4)])  # more than 64 sequences
def test_workgroups_by_length(B, Hq, Hkv, r, L_cap, kind, chunks, append):
    import torch
    from paper_2506_02572_amd import hata
    print(f"[encode_score] B={B} Hq={Hq} Hkv={Hkv} r={r} L_cap={L_cap} {kind} append={append}", flush=True)
    lens, k_max = batch(kind, B, L_cap), 100
    ctx = hata.Context(B, Hq, Hkv, 128, r, L_cap, k_max, shared_device=True)
    most = chunks_of_a_workgroup(ctx, B, Hq, Hkv, r)
    assert most > 1
    _, chunk, n_chunks = ctx.hata_step_plan(B)
    assert chunks_by_length(n_chunks, chunk, most, [min(n, L_cap) for n in lens]) == chunks
    g = torch.Generator(device="cuda").manual_seed(B + Hq + r)
    K, V = (torch.randn((B, Hkv, L_cap, 128), dtype=torch.bfloat16, device="cuda", generator=g) for _ in range(2))
    q = torch.randn((B, Hq, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    W = torch.randn((Hkv, 128, r), dtype=torch.float32, device="cuda", generator=g)
    codes = torch.randint(-2**31, 2**31 - 1, (B, Hkv, L_cap, r // 32), dtype=torch.int32, device="cuda", generator=g)
    seq = torch.tensor(lens, dtype=torch.int32, device="cuda")
    kb = torch.tensor([min(n, k_max - b % 7) for b, n in enumerate(lens)], dtype=torch.int32, device="cuda")
    want = codes.clone()
    if append:
        there = ((seq > 0) & (seq <= L_cap)).to(torch.int32)
        ctx.hata_encode_keys(K, W, torch.clamp(seq - 1, 0, L_cap - 1), there, B, 1, want)
    out = torch.empty((B, Hq, 128), dtype=torch.bfloat16, device="cuda")
    for _ in range(2):
        ctx.hata_decode_step(q, K, V, W, codes, seq, kb, B, append, 1.0 / math.sqrt(128), out)
    torch.cuda.synchronize()
    qcodes, scores, idx = (t.clone() for t in ctx.hata_step_buffers())
    want_q, want_s, want_i = torch.zeros_like(qcodes), torch.zeros_like(scores).view(B, Hkv, L_cap), torch.zeros_like(idx).view(B, Hkv, k_max)
    ctx.hata_encode_query(q, W, B, want_q)
    ctx.hata_hamming_score(want_q, want, seq, B, want_s)
    ctx.hata_topk(want_s, seq, kb, B, want_i)
    torch.cuda.synchronize()
    assert torch.equal(codes, want) and torch.equal(qcodes, want_q)
    scores = scores.view(want_s.shape)
    for b, n in enumerate(lens):
        assert torch.equal(scores[b, :, :min(n, L_cap)], want_s[b, :, :min(n, L_cap)]), b
    assert torch.equal(idx.view(want_i.shape), want_i)
    ctx.close()
