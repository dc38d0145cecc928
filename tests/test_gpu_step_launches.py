"""What the single-launch step keeps between launches: after one that gave up a wait, and between captured and eager ones."""
import ctypes
import functools
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hata_oracle as O
from paper_2506_02572_amd import synth
from tests import harness as H

SCALE = 1.0 / math.sqrt(128)


def make_case(r, heads, seq, k_max):
    (Hq, Hkv), B, L = heads, len(seq), max(seq)
    rng = np.random.default_rng(L + r)
    seq, k = np.array(seq, np.int32), np.array([max(1, k_max >> b) for b in range(B)], np.int32)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L, 128))) for _ in range(2))
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    codes = rng.integers(0, 2**32, (B, Hkv, L, r // 32), dtype=np.uint32)
    queries = [synth.round_to_bf16_bits(rng.standard_normal((B, Hq, 128))) for _ in range(4)]
    refs = [O.decode_step(q, K, V, W, codes.copy(), seq, k, k_max, SCALE, append=False) for q in queries]
    return seq, k, K, V, W, codes, queries, refs


@pytest.mark.parametrize("r,heads,seq,k_max,chunk", [(128, (8, 2), (9000, 5000, 1000), 200, 1024), (256, (8, 1), (70000, 3000), 500, 1024),
                                                     (64, (16, 2), (30000, 9000), 90, 1024), (128, (16, 4), (40000, 17000), 300, 16384)])
def test_step_after_one_that_gave_up(r, heads, seq, k_max, chunk):
    """No call of hata_check between them.  Two contexts over one workspace, so that host-side counts are the same in both
    launches, as in replays of one graph: the second launch is right, with queries of its own."""
    import torch
    from paper_2506_02572_amd import hata
    print(f"[launches] r={r} heads={heads} seq={seq} chunk={chunk}", flush=True)
    (Hq, Hkv), B, L = heads, len(seq), max(seq)
    seq, k, K, V, W, codes, queries, refs = make_case(r, heads, seq, k_max)
    Kd, Vd, Wd, cd, sd, kd = (H.to_dev(x) for x in (K, V, W, codes, seq, k))
    out = torch.zeros((B, Hq, 128), dtype=torch.int16, device="cuda")
    out32 = torch.zeros((B, Hq, 128), dtype=torch.float32, device="cuda")
    for turn in range(4):
        ctx = hata.Context(B, Hq, Hkv, 128, r, L, k_max, chunk=chunk)
        second = ctypes.c_void_p(None)
        rc = ctx._lib.hata_create_tuned(ctypes.byref(second), ctypes.byref(ctx.cfg), ctypes.byref(ctx.tuning),
                                        ctypes.c_void_p(ctx._ws_ptr), ctx.workspace_bytes)
        assert rc == 0 and ctx.hata_step_plan(B)[:2] == (1, chunk)
        first = ctx._h
        ctx.hata_set_wait_limit(1)
        for _ in range(1 + turn // 2):
            ctx.hata_decode_step(H.to_dev(queries[turn]), Kd, Vd, Wd, cd, sd, kd, B, False, SCALE, out, out32)
        assert np.any(np.isnan(H.to_host(out32))), "a wait bound of one poll was expected to be given up"
        ctx._h = second
        try:
            if turn % 2:  # the selection alone first
                idx = torch.zeros((B, Hkv, k_max), dtype=torch.int32, device="cuda")
                ctx.hata_select_step(H.to_dev(queries[3 - turn]), None, Wd, cd, sd, kd, B, False, idx)
                assert np.array_equal(H.to_host(idx), refs[3 - turn]["idx"])
            for j in (1, 2):
                n = (turn + j) % 4
                ctx.hata_decode_step(H.to_dev(queries[n]), Kd, Vd, Wd, cd, sd, kd, B, False, SCALE, out, out32)
                torch.cuda.synchronize()
                assert np.array_equal(H.to_host(ctx.hata_step_buffers()[2]), refs[n]["idx"])
                H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), refs[n]["out"], "behind a give-up")
            with pytest.raises(hata.HataError, match="gave up"):
                ctx.hata_check()
        finally:
            ctx._lib.hata_destroy(first)
            ctx.close()


def test_replays_beside_eager_steps_of_other_batches():
    """A graph of a step for two of three sequences, replayed between eager steps of one, two and three sequences and one that
    gives up: units that sit launches out keep a count of their own."""
    import torch
    from paper_2506_02572_amd import hata
    r, heads, k_max, chunk, B = 128, (8, 2), 150, 1024, 3
    seq, k, K, V, W, codes, queries, refs = make_case(r, heads, (9000, 7000, 3000), k_max)
    ctx = hata.Context(B, heads[0], heads[1], 128, r, int(seq.max()), k_max, chunk=chunk)
    Kd, Vd, Wd, cd, sd, kd = (H.to_dev(x) for x in (K, V, W, codes, seq, k))
    qd = H.to_dev(queries[0])
    out = torch.zeros((B, heads[0], 128), dtype=torch.int16, device="cuda")
    out32 = torch.zeros((B, heads[0], 128), dtype=torch.float32, device="cuda")

    def step(n):
        ctx.hata_decode_step(qd, Kd, Vd, Wd, cd, sd, kd, n, False, SCALE, out, out32)

    def check(n, query):
        torch.cuda.synchronize()
        assert np.array_equal(H.to_host(ctx.hata_step_buffers()[2])[:n], refs[query]["idx"][:n])
        H.check_attention(H.to_host(out32)[:n], H.to_host(out, np.uint16)[:n], refs[query]["out"][:n], "replay")

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(2)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step(2)
    for turn, (eager, gives_up) in enumerate([(3, False), (1, False), (3, True), (2, True), (1, True), (3, False)]):
        query = turn % 4
        qd.copy_(H.to_dev(queries[query]))
        torch.cuda.synchronize()
        ctx.hata_set_wait_limit(1 if gives_up else 0)
        step(eager)
        if not gives_up:
            check(eager, query)
        ctx.hata_set_wait_limit(0)
        for again in (1, 2):
            query = (turn + again) % 4
            qd.copy_(H.to_dev(queries[query]))
            torch.cuda.synchronize()
            out32.fill_(7.0)
            g.replay()
            check(2, query)
            assert torch.all(out32[2] == 7.0)
    step(3)
    check(3, query)
    with pytest.raises(hata.HataError, match="gave up"):
        ctx.hata_check()
    step(3)
    check(3, query)
    ctx.hata_check()
    ctx.close()


@pytest.mark.parametrize("B,Hkv,L_cap", [(16, 8, 32768), (8, 8, 65536), (4, 8, 131072), (1, 32, 131072)])
def test_chunk_goes_by_residency_alone(B, Hkv, L_cap):
    """A batch that is resident at 4096 keys a workgroup stays at that: how full its caches are only the device knows."""
    from paper_2506_02572_amd import hata
    print(f"[launches] chunk of {B} caches of {L_cap} rows", flush=True)
    ctx = hata.Context(B, 32, Hkv, 128, 128, L_cap, 512)
    assert ctx.hata_step_plan(B) == (1, 4096, L_cap // 4096) and ctx.hata_step_sub_batches(B) == 1
    ctx.close()


def test_plan_with_more_chunks_than_the_step_runs_with():
    """1.1M rows are 269 chunks of the plan and fewer of the single-launch step: the same rows as three launches select."""
    import torch
    from paper_2506_02572_amd import hata
    L, Hkv, G, r, k_max = 1_100_000, 2, 4, 64, 700
    print(f"[launches] {L} rows", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    K = torch.randn((1, Hkv, L, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    q = torch.randn((1, Hkv * G, 128), dtype=torch.bfloat16, device="cuda", generator=g)
    W = torch.randn((Hkv, 128, r), device="cuda", generator=g)
    codes = torch.randint(-2**31, 2**31 - 1, (1, Hkv, L, r // 32), dtype=torch.int32, device="cuda", generator=g)
    k = H.to_dev(np.array([k_max], np.int32))
    ctx = hata.Context(1, Hkv * G, Hkv, 128, r, L, k_max)
    assert -(-L // 4096) > 256 >= ctx.hata_step_plan(1)[2] > 1 and ctx.hata_step_plan(1)[0] == 1
    for rows in (L, L - 70_001, 5):
        seq = H.to_dev(np.array([rows], np.int32))
        got = []
        for mode in (0, 3):
            ctx.hata_set_step_mode(mode)
            out = torch.zeros((1, Hkv * G, 128), dtype=torch.float32, device="cuda")
            for _ in range(2):
                ctx.hata_decode_step(q, K, K, W, codes, seq, k, 1, False, SCALE, torch.empty_like(q), out)
            ctx.hata_check()
            got.append((H.to_host(ctx.hata_step_buffers()[2]).copy(), out))
        assert np.array_equal(got[0][0], got[1][0])
        # (fp32 sums in another order, weights of 16 bits or more: hata_attn_core.h)
        assert torch.allclose(got[0][1], got[1][1], rtol=1e-3, atol=1e-4)
    ctx.close()


@pytest.mark.parametrize("form,heads,r", [
    (f, h, r) for f in ("waits", "waits_large_chunks", "waits_one_grid", "paged", "three_launches", "unit")
    for h, r in (((4, 4), 128), ((10, 2), 64), ((16, 2), 256), ((16, 1), 128))
    if f != "unit" or h != (16, 1)])  # (no workgroup per unit for groups of sixteen)
def test_empty_sequences_and_budgets_in_every_form(form, heads, r):
    """Sequences without rows and budgets of none beside others, twice over: the second step finds what the first one left."""
    import torch
    from paper_2506_02572_amd import hata
    from tests.test_gpu_paged import make_table, scatter
    (Hq, Hkv), k_max, page_rows = heads, 90, 64
    print(f"[launches] empty, {form} heads={heads} r={r}", flush=True)
    seq, k = np.array([0, 3900, 1, 2050, 0, 1024], np.int32), np.array([5, 0, 7, 90, 0, 3], np.int32)
    B, L = len(seq), 3900
    rng = np.random.default_rng(r + Hq)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L, 128))) for _ in range(2))
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    codes = rng.integers(0, 2**32, (B, Hkv, L, r // 32), dtype=np.uint32)
    ctx = hata.Context(B, Hq, Hkv, 128, r, L, k_max, chunk={"waits_large_chunks": 16384, "unit": 0, "three_launches": 0}.get(form, 1024))
    ctx.hata_set_step_mode({"waits_one_grid": 1, "three_launches": 3}.get(form, 0))
    launches, _, chunks = ctx.hata_step_plan(B)
    assert launches == (3 if form == "three_launches" else 1) and (chunks == 1) == (form in ("unit", "waits_large_chunks"))
    cache = [H.to_dev(x) for x in (K, V, W, codes)]
    call = ctx.hata_decode_step
    if form == "paged":
        table, max_blocks, n_pages, blocks = make_table(rng, seq, page_rows)
        pools = []
        for x in (K, V, codes):
            pool = np.zeros((n_pages, Hkv, page_rows, x.shape[-1]), x.dtype)
            scatter(pool, x, table, blocks, page_rows, seq)
            pools.append(H.to_dev(pool))
        cache = [pools[0], pools[1], cache[2], pools[2], H.to_dev(table), max_blocks, page_rows, n_pages]
        call = ctx.hata_decode_step_paged
    out = torch.zeros((B, Hq, 128), dtype=torch.int16, device="cuda")
    out32 = torch.zeros((B, Hq, 128), dtype=torch.float32, device="cuda")
    for turn, order in enumerate((np.arange(B), np.arange(B), np.arange(B)[::-1])):
        # (the lengths change places in the last turn: units that had rows have none, and the other way round)
        s2, k2 = (seq, k) if form == "paged" else (seq[order], k[order])
        q = synth.round_to_bf16_bits(rng.standard_normal((B, Hq, 128)))
        ref = O.decode_step(q, K, V, W, codes.copy(), s2, k2, k_max, SCALE, append=False)
        out32.fill_(float("nan"))
        call(H.to_dev(q), *cache, H.to_dev(s2), H.to_dev(k2), B, False, SCALE, out, out32)
        ctx.hata_check()
        assert np.array_equal(H.to_host(ctx.hata_step_buffers()[0], np.uint32), ref["qcodes"])
        assert np.array_equal(H.to_host(ctx.hata_step_buffers()[2]), ref["idx"])
        H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), ref["out"], form)
    ctx.close()


@functools.lru_cache(maxsize=1)
def make_unlike_chunks(heads, r, seq, k_max, budgets):
    """Codes whose chunks of 1024 keys have a share of the query's bits of their own, so that the distributions hardly
    overlap (every third sequence: the same share everywhere)."""
    (Hq, Hkv), B, L = heads, len(seq), max(seq)
    rng = np.random.default_rng(L + r)
    K = synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L, 128), dtype=np.float32))
    V = np.roll(K, 1, axis=3)
    W = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    q = synth.round_to_bf16_bits(np.repeat(rng.standard_normal((B, Hkv, 1, 128)), Hq // Hkv, 2).reshape(B, Hq, 128))
    one = np.ones(B, np.int32)
    qc = O.decode_step(q, K[:, :, :1], V[:, :, :1], W, np.zeros((B, Hkv, 1, r // 32), np.uint32), one, one, 1, SCALE,
                       append=False)["qcodes"].reshape(B, Hkv, Hq // Hkv, r // 32)[:, :, :1]
    share = rng.integers(0, 9, (B, -(-L // 1024)))
    share[::3] = 4
    share = np.repeat(share, 1024, 1)[:, None, :L, None]
    flips = rng.integers(0, 2**32, (B, Hkv, L, r // 32), dtype=np.uint32)
    for i in range(3):  # a bit flipped with probability 1/2, 1/4 .. 1/16, or kept with it
        flips &= np.where(share % 4 > i, rng.integers(0, 2**32, flips.shape, dtype=np.uint32), np.uint32(0xffffffff))
    codes = qc ^ np.where(share >= 5, ~flips, flips)
    n = np.array(seq, np.int32)
    refs = [O.decode_step(q, K, V, W, codes.copy(), n, np.full(B, k, np.int32), k_max, SCALE, append=False) for k in budgets]
    return rng, q, K, V, W, codes, refs


@pytest.mark.parametrize("heads,r", [((4, 1), 128), ((8, 1), 256), ((2, 2), 64)])
@pytest.mark.parametrize("seq", [(1025, 1024 + 255, 1024 + 256, 2049), (13 * 1024 + 2, 25 * 1024 + 1, 33 * 1024 + 3), (64 * 1024 + 2, 65 * 1024 + 200, 64 * 1024)])
@pytest.mark.parametrize("form", ["waits", "waits_large_chunks", "paged", "three_launches", "three_launches_pieces"])
def test_last_chunk_of_a_few_keys(form, heads, r, seq):
    """It goes by the estimate of the chunk before; that one's keys are like the others' or nothing like them."""
    import torch
    from paper_2506_02572_amd import hata
    from tests.test_gpu_paged import make_table, scatter
    (Hq, Hkv), B, L, k_max, page_rows, budgets = heads, len(seq), max(seq), 700, 64, (1, 150, 700)
    print(f"[launches] few keys, {form} heads={heads} r={r} seq={seq}", flush=True)
    rng, q, K, V, W, codes, refs = make_unlike_chunks(heads, r, seq, k_max, budgets)
    seq = np.array(seq, np.int32)
    ctx = hata.Context(B, Hq, Hkv, 128, r, L, k_max, chunk=16384 if form == "waits_large_chunks" else 1024,
                       attn_rows=16 if form == "three_launches_pieces" else 0)
    ctx.hata_set_step_mode(3 if form.startswith("three") else 0)
    assert ctx.hata_step_plan(B)[0] == (3 if form.startswith("three") else 1)
    cache = [H.to_dev(x) for x in (K, V, W, codes)]
    call = ctx.hata_decode_step
    if form == "paged":
        table, max_blocks, n_pages, blocks = make_table(rng, seq, page_rows)
        pools = []
        for x in (K, V, codes):
            pool = np.zeros((n_pages, Hkv, page_rows, x.shape[-1]), x.dtype)
            scatter(pool, x, table, blocks, page_rows, seq)
            pools.append(H.to_dev(pool))
        cache = [pools[0], pools[1], cache[2], pools[2], H.to_dev(table), max_blocks, page_rows, n_pages]
        call = ctx.hata_decode_step_paged
    out = torch.zeros((B, Hq, 128), dtype=torch.int16, device="cuda")
    out32 = torch.zeros((B, Hq, 128), dtype=torch.float32, device="cuda")
    for budget, ref in zip(budgets, refs):
        call(H.to_dev(q), *cache, H.to_dev(seq), H.to_dev(np.full(B, budget, np.int32)), B, False, SCALE, out, out32)
        ctx.hata_check()
        assert np.array_equal(H.to_host(ctx.hata_step_buffers()[2]), ref["idx"])
        H.check_attention(H.to_host(out32), H.to_host(out, np.uint16), ref["out"], form)
    ctx.close()
