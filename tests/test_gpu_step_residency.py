"""Grids of the single-launch step just above what fits the device, at the sizes where that is hard to tell -- a workgroup's LDS just below a third of
a compute unit's, registers of a kernel that asks for four workgroups at most --: the step finishes, and selects what the stage calls select."""
import math

import pytest

pytestmark = pytest.mark.gpu


def selection(torch, hata, B, Hq, Hkv, r, L_cap, k, q, W, codes, seq, kb):
    """By the stage calls; codes [B, Hkv, L_cap, r / 32]."""
    ctx = hata.Context(B, Hq, Hkv, 128, r, L_cap, k)
    qcodes = torch.zeros((B, Hq, r // 32), dtype=torch.int32, device="cuda")
    scores = torch.zeros((B, Hkv, L_cap), dtype=torch.int16, device="cuda")
    idx = torch.zeros((B, Hkv, k), dtype=torch.int32, device="cuda")
    ctx.hata_encode_query(q, W, B, qcodes)
    ctx.hata_hamming_score(qcodes, codes, seq, B, scores)
    ctx.hata_topk(scores, seq, kb, B, idx)
    torch.cuda.synchronize()
    ctx.close()
    return idx


@pytest.mark.parametrize("Hq,r,L,paged", [
    (32, 128, 40529, True),   # 8192 keys a workgroup, 53840 bytes: 640 workgroups, 512 of them resident
    (32, 128, 40960, True), (64, 64, 40529, False), (32, 128, 40529, False),
    (8, 64, 40529, False), (16, 32, 40529, False), (8, 32, 36865, True), (16, 64, 38000, True),  # 85 registers or fewer: 1280 workgroups, 1024 resident
    (16, 64, 77000, True), (16, 32, 77000, True)])                                              # both (16384 keys a workgroup, or 4096)
def test_grid_above_what_is_resident(Hq, r, L, paged):
    import torch
    from paper_2506_02572_amd import hata
    print(f"[residency] Hq={Hq} r={r} L={L} paged={paged}", flush=True)
    B, Hkv, k, P, scale = 16, 8, 100, 64, 1.0 / math.sqrt(128)
    L_cap = -(-L // P) * P
    g = torch.Generator(device="cuda").manual_seed(L + r)
    q = torch.randn((B, Hq, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    W = torch.randn((Hkv, 128, r), dtype=torch.float32, device="cuda", generator=g)
    seq = torch.full((B,), L, dtype=torch.int32, device="cuda")
    kb = torch.full((B,), k, dtype=torch.int32, device="cuda")
    out = torch.zeros((B, Hq, 128), dtype=torch.bfloat16, device="cuda")
    n_pages = L_cap // P
    one = torch.randint(-2**31, 2**31 - 1, (Hkv, L_cap, r // 32), dtype=torch.int32, device="cuda", generator=g)
    codes = one.expand(B, Hkv, L_cap, r // 32).contiguous()
    want = selection(torch, hata, B, Hq, Hkv, r, L_cap, k, q, W, codes, seq, kb)
    ctx = hata.Context(B, Hq, Hkv, 128, r, L_cap, k)
    if paged:  # all sequences read the same pages
        K, V = (torch.randn((n_pages, Hkv, P, 128), dtype=torch.bfloat16, device="cuda", generator=g) for _ in range(2))
        pages = torch.randperm(n_pages, device="cuda", generator=g)
        pool = torch.empty((n_pages, Hkv, P, r // 32), dtype=torch.int32, device="cuda")
        pool[pages] = one.view(Hkv, n_pages, P, r // 32).transpose(0, 1)
        table = pages.to(torch.int32).expand(B, n_pages).contiguous()
        ctx.hata_decode_step_paged(q, K, V, W, pool, table, n_pages, P, n_pages, seq, kb, B, False, scale, out)
    else:
        K, V = (torch.randn((B, Hkv, L_cap, 128), dtype=torch.bfloat16, device="cuda", generator=g) for _ in range(2))
        ctx.hata_decode_step(q, K, V, W, codes, seq, kb, B, False, scale, out)
    ctx.hata_check()  # raises if a workgroup gave up waiting
    assert torch.equal(ctx.hata_step_buffers()[2].view(want.shape), want)
    assert bool(torch.isfinite(out.float()).all())
    ctx.close()
