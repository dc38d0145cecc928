"""The step with a workgroup per (sequence, KV head) unit at the edges of its ranges, against the oracle."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hata_oracle as O
from paper_2506_02572_amd import synth
from tests import harness as H
from tests.test_gpu_paged import make_table, scatter

SCALE = 1.0 / math.sqrt(128)


@pytest.mark.parametrize("L_cap", [1, 3, 64, 1023, 1025, 4095, 4096, 4097, 8191, 8192])
@pytest.mark.parametrize("heads,r", [((1, 1), 32), ((2, 1), 64), ((4, 1), 128), ((5, 1), 256), ((16, 2), 128), ((8, 1), 256), ((3, 3), 128)])
@pytest.mark.parametrize("ties", [False, True])
def test_unit_step(L_cap, heads, r, ties):
    import torch
    from paper_2506_02572_amd import hata
    (Hq, Hkv), B = heads, 3
    print(f"[unit] L_cap={L_cap} heads={heads} r={r} ties={ties}", flush=True)
    rng = np.random.default_rng(L_cap + r + Hq)
    seq = np.array([L_cap, max(1, L_cap - 5), max(1, L_cap // 2)], np.int32)  # (an empty sequence has no row to append)
    k_max = max(1, min(L_cap // 3, 2_200_000 // L_cap))  # (larger budgets of so few units go to several workgroups a unit)
    k = np.array([max(1, min(L_cap // 50, k_max)), k_max, 0 if L_cap < 100 else 40], np.int32)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L_cap, 128))) for _ in range(2))
    q = synth.round_to_bf16_bits(rng.standard_normal((B, Hq, 128)))
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    codes = rng.integers(0, 2**32, (B, Hkv, L_cap, r // 32), dtype=np.uint32)
    if ties:
        codes = codes[:, :, rng.integers(0, min(2, L_cap), L_cap)]
    want = codes.copy()
    ref = O.decode_step(q, K, V, W, want, seq, k, k_max, SCALE, append=True)
    ctx = hata.Context(B, Hq, Hkv, 128, r, L_cap, k_max, shared_device=True)
    assert ctx.hata_step_plan(B)[0] == 1 and ctx.hata_step_plan(B)[2] == 1
    ctx.hata_keep_step_scores(True)
    cd = H.to_dev(codes)
    out = torch.full((B, Hq, 128), -1, dtype=torch.int16, device="cuda")
    out32 = torch.full((B, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
    ctx.hata_decode_step(H.to_dev(q), H.to_dev(K), H.to_dev(V), H.to_dev(W), cd, H.to_dev(seq), H.to_dev(k), B, True, SCALE, out, out32)
    torch.cuda.synchronize()
    qc, sc, ix = ctx.hata_step_buffers()
    assert np.array_equal(H.to_host(qc, np.uint32), ref["qcodes"])
    assert np.array_equal(H.to_host(cd, np.uint32), want)
    for b in range(B):
        assert np.array_equal(H.to_host(sc, np.uint16)[b, :, :seq[b]].astype(np.int32), ref["scores"][b, :, :seq[b]])
    assert np.array_equal(H.to_host(ix), ref["idx"])
    H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), ref["out"], "unit step")
    ctx.close()


@pytest.mark.parametrize("units,L_cap,page_rows", [((32, 4), 8192, 0), ((32, 4), 8192, 16), ((32, 8), 16384, 0), ((32, 8), 16384, 256), ((2, 2), 4000, 64)])
def test_unit_step_of_many_units(units, L_cap, page_rows):
    """Own device: the form is taken by the number of units; its outputs against those of workgroups that share units."""
    import torch
    from paper_2506_02572_amd import hata
    (B, Hkv), r, k_max = units, 64, 200
    print(f"[unit] {units} L_cap={L_cap} page_rows={page_rows}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(L_cap)
    K, V = (torch.randn((B, Hkv, L_cap, 128), dtype=torch.bfloat16, device="cuda", generator=g) for _ in range(2))
    q = torch.randn((B, Hkv * 2, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    W = torch.randn((Hkv, 128, r), device="cuda", generator=g)
    codes = torch.randint(-2**31, 2**31 - 1, (B, Hkv, L_cap, r // 32), dtype=torch.int32, device="cuda", generator=g)
    rng = np.random.default_rng(B)
    seq = rng.integers(L_cap // 2, L_cap, B).astype(np.int32)
    k = rng.integers(1, k_max, B).astype(np.int32)
    got = []
    for shared_units in (False, True):
        ctx = hata.Context(B, Hkv * 2, Hkv, 128, r, L_cap, k_max, chunk=4096 if shared_units else 0)
        assert (ctx.hata_step_plan(B)[2] == 1) == (not shared_units or L_cap <= 4096)
        cd, out, out32 = codes.clone(), torch.zeros_like(q), torch.zeros(q.shape, dtype=torch.float32, device="cuda")
        args = [q, K, V, W, cd]
        if page_rows and not shared_units:
            table, max_blocks, n_pages, blocks = make_table(rng, seq, page_rows)
            pools = []
            for x, dt in ((K.view(torch.int16), np.int16), (V.view(torch.int16), np.int16), (cd, np.int32)):
                pool = np.zeros((n_pages, Hkv, page_rows, x.shape[-1]), dt)
                scatter(pool, H.to_host(x), table, blocks, page_rows, seq)
                pools.append(H.to_dev(pool))
            ctx.hata_decode_step_paged(q, pools[0], pools[1], W, pools[2], H.to_dev(table), max_blocks, page_rows, n_pages,
                                       H.to_dev(seq), H.to_dev(k), B, True, SCALE, out, out32)
        else:
            ctx.hata_decode_step(*args, H.to_dev(seq), H.to_dev(k), B, True, SCALE, out, out32)
        ctx.hata_check()
        got.append((H.to_host(ctx.hata_step_buffers()[2]).copy(), out32))
        ctx.close()
    assert np.array_equal(got[0][0], got[1][0])
    # (fp32 sums in another order, weights of 16 bits or more: hata_attn_core.h)
    assert torch.allclose(got[0][1], got[1][1], rtol=1e-3, atol=1e-4)


@pytest.mark.parametrize("L_cap,Hkv,G,r,k_max,B,shared,unit", [
    (4096, 8, 4, 128, 64, 1, False, True), (4096, 8, 4, 128, 2048, 1, False, False), (4096, 8, 1, 128, 1024, 1, False, True),
    (4096, 8, 4, 128, 2048, 24, False, True), (8192, 8, 4, 128, 256, 16, False, True), (8192, 8, 4, 128, 2048, 16, False, False),
    (8192, 8, 4, 128, 200, 1, True, True), (8192, 8, 4, 128, 2048, 1, True, False), (8192, 8, 4, 256, 384, 1, True, False),
    (16384, 8, 4, 128, 2048, 32, False, True), (16384, 8, 4, 128, 512, 16, True, True)])
def test_budgets_a_unit_workgroup_takes(L_cap, Hkv, G, r, k_max, B, shared, unit):
    """A compute unit alone gathers rows slowly: budgets that are large for so few units go to several workgroups a unit."""
    from paper_2506_02572_amd import hata
    print(f"[unit] rule L_cap={L_cap} units={B * Hkv} G={G} r={r} k_max={k_max} shared={shared}", flush=True)
    ctx = hata.Context(B, Hkv * G, Hkv, 128, r, L_cap, k_max, shared_device=shared)
    launches, _, chunks = ctx.hata_step_plan(B)
    assert ((launches, chunks) == (1, 1)) == unit
    ctx.close()


@pytest.mark.parametrize("L_cap", [700, 5000])
def test_scores_of_a_shared_device(L_cap):
    """A context of a shared device leaves the scores in the workspace without being asked, whatever form its steps take."""
    import torch
    from paper_2506_02572_amd import hata
    B, Hq, Hkv, r, k_max = 2, 4, 1, 64, 40
    print(f"[unit] scores of a shared device, L_cap={L_cap}", flush=True)
    rng = np.random.default_rng(L_cap)
    seq, k = np.array([L_cap, L_cap // 2], np.int32), np.array([k_max, 9], np.int32)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L_cap, 128))) for _ in range(2))
    q = synth.round_to_bf16_bits(rng.standard_normal((B, Hq, 128)))
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    codes = rng.integers(0, 2**32, (B, Hkv, L_cap, r // 32), dtype=np.uint32)
    ref = O.decode_step(q, K, V, W, codes.copy(), seq, k, k_max, SCALE, append=False)
    out = torch.zeros((B, Hq, 128), dtype=torch.int16, device="cuda")
    dev = [H.to_dev(x) for x in (q, K, V, W, codes, seq, k)]
    for launches in (1, 3):
        ctx = hata.Context(B, Hq, Hkv, 128, r, L_cap, k_max, shared_device=True)
        if launches == 3:
            ctx.hata_set_step_mode(3)
        assert ctx.hata_step_plan(B)[0] == launches
        scores = ctx.hata_step_buffers()[1]
        scores.fill_(-1)
        ctx.hata_decode_step(*dev, B, False, SCALE, out)
        torch.cuda.synchronize()
        for b in range(B):
            assert np.array_equal(H.to_host(scores, np.uint16)[b, :, :seq[b]].astype(np.int32), ref["scores"][b, :, :seq[b]])
            assert np.all(H.to_host(scores, np.uint16)[b, :, seq[b]:] == 0xffff)
        ctx.close()


@pytest.mark.parametrize("mode", [0, 1, 3])
@pytest.mark.parametrize("L_cap", [3000, 7000])
def test_paged_step_knows_no_modes(mode, L_cap):
    """The block-table step of a short cache takes a workgroup per unit, whatever mode the other layout was given: nothing in
    it waits, so one poll is enough (the form with waits would give up)."""
    import torch
    from paper_2506_02572_amd import hata
    B, Hq, Hkv, r, k_max, page_rows = 2, 8, 2, 128, 96, 64
    print(f"[unit] paged, mode={mode} L_cap={L_cap}", flush=True)
    rng = np.random.default_rng(L_cap)
    seq, k = np.array([L_cap, L_cap - 100], np.int32), np.array([k_max, 50], np.int32)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L_cap, 128))) for _ in range(2))
    q = synth.round_to_bf16_bits(rng.standard_normal((B, Hq, 128)))
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    codes = rng.integers(0, 2**32, (B, Hkv, L_cap, r // 32), dtype=np.uint32)
    ref = O.decode_step(q, K, V, W, codes.copy(), seq, k, k_max, SCALE, append=False)
    table, max_blocks, n_pages, blocks = make_table(rng, seq, page_rows)
    pools = []
    for x in (K, V, codes):
        pool = np.zeros((n_pages, Hkv, page_rows, x.shape[-1]), x.dtype)
        scatter(pool, x, table, blocks, page_rows, seq)
        pools.append(H.to_dev(pool))
    ctx = hata.Context(B, Hq, Hkv, 128, r, L_cap, k_max, shared_device=True)
    ctx.hata_set_step_mode(mode)
    ctx.hata_set_wait_limit(1)
    out = torch.zeros((B, Hq, 128), dtype=torch.int16, device="cuda")
    out32 = torch.zeros((B, Hq, 128), dtype=torch.float32, device="cuda")
    ctx.hata_decode_step_paged(H.to_dev(q), pools[0], pools[1], H.to_dev(W), pools[2], H.to_dev(table), max_blocks, page_rows,
                               n_pages, H.to_dev(seq), H.to_dev(k), B, False, SCALE, out, out32)
    ctx.hata_check()
    assert np.array_equal(H.to_host(ctx.hata_step_buffers()[2]), ref["idx"])
    H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), ref["out"], "paged unit step")
    ctx.close()


@pytest.mark.parametrize("L_cap", [8193, 12000, 16384])
@pytest.mark.parametrize("G,r", [(1, 128), (4, 256), (5, 128), (8, 256), (8, 128), (4, 128)])
@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("page_rows", [0, 64])
def test_unit_step_of_long_caches(L_cap, G, r, ties, page_rows):
    """Sixteen keys a thread, in both layouts: 128 sequences over the rows of one cache, two of them against the oracle."""
    import torch
    from paper_2506_02572_amd import hata
    B, k_max, look = 128, 500, [0, 127]
    print(f"[unit] long L_cap={L_cap} G={G} r={r} ties={ties} page_rows={page_rows}", flush=True)
    rng = np.random.default_rng(L_cap + G + r)
    seq, k = rng.integers(1, L_cap + 1, B).astype(np.int32), rng.integers(0, k_max + 1, B).astype(np.int32)
    seq[look], k[look] = (L_cap, L_cap - 1030), (k_max, 77)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((1, 1, L_cap, 128))) for _ in range(2))
    q = synth.round_to_bf16_bits(rng.standard_normal((B, G, 128)))
    W = rng.standard_normal((1, 128, r)).astype(np.float32)
    codes = rng.integers(0, 2**32, (1, 1, L_cap, r // 32), dtype=np.uint32)
    if ties:
        codes = codes[:, :, rng.integers(0, 2, L_cap)]
    ctx = hata.Context(B, G, 1, 128, r, L_cap, k_max, kv_strides=(0, 0, 128), shared_device=True)
    assert ctx.hata_step_plan(B)[0] == 1 and ctx.hata_step_plan(B)[2] == 1
    ctx.hata_keep_step_scores(True)
    out = torch.zeros((B, G, 128), dtype=torch.int16, device="cuda")
    out32 = torch.full((B, G, 128), float("nan"), dtype=torch.float32, device="cuda")
    if page_rows:
        table, max_blocks, n_pages, blocks = make_table(rng, [L_cap], page_rows)
        pools = []
        for x in (K, V, codes):
            pool = np.zeros((n_pages, 1, page_rows, x.shape[-1]), x.dtype)
            scatter(pool, x, table, blocks, page_rows, [L_cap])
            pools.append(H.to_dev(pool))
        ctx.hata_decode_step_paged(H.to_dev(q), pools[0], pools[1], H.to_dev(W), pools[2], H.to_dev(np.repeat(table, B, 0)), max_blocks,
                                   page_rows, n_pages, H.to_dev(seq), H.to_dev(k), B, False, SCALE, out, out32)
    else:
        ctx.hata_decode_step(H.to_dev(q), H.to_dev(K), H.to_dev(V), H.to_dev(W), H.to_dev(np.repeat(codes, B, 0)), H.to_dev(seq),
                             H.to_dev(k), B, False, SCALE, out, out32)
    torch.cuda.synchronize()
    two = [np.repeat(x, 2, 0) for x in (K, V, codes)]
    ref = O.decode_step(q[look], two[0], two[1], W, two[2], seq[look], k[look], k_max, SCALE, append=False)
    qc, sc, ix = ctx.hata_step_buffers()
    assert np.array_equal(H.to_host(qc, np.uint32)[look], ref["qcodes"])
    for i, b in enumerate(look):
        assert np.array_equal(H.to_host(sc[b], np.uint16)[:, :seq[b]].astype(np.int32), ref["scores"][i, :, :seq[b]])
    assert np.array_equal(H.to_host(ix)[look], ref["idx"])
    H.check_attention(H.to_host(out32)[look], H.to_host(out, np.uint16)[look], ref["out"], "long unit step")
    assert not torch.isnan(out32).any()
    ctx.close()
