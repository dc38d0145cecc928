"""The single-launch step's threshold search where the chunks of a unit differ, against the oracle."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hata_oracle as O
from paper_2506_02572_amd import synth
from tests import harness as H


@pytest.mark.parametrize("r,heads,L,chunk", [(128, (4, 1), 5000, 1024), (256, (8, 1), 9000, 1024), (256, (4, 2), 70000, 1024),
                                             (32, (1, 1), 3000, 1024), (64, (5, 1), 40000, 16384), (128, (16, 2), 12289, 4096)])
@pytest.mark.parametrize("kind", ["one_near", "one_far", "staircase", "two_values"])
def test_threshold_of_unequal_chunks(r, heads, L, chunk, kind):
    """Every chunk estimates the threshold from its own keys: here the estimates are off by up to the whole range of scores."""
    compare_steps(r, heads, L, chunk, kind)


@pytest.mark.parametrize("r,heads,chunks", [(128, (64, 8), 12), (128, (64, 8), 13), (64, (8, 8), 24), (64, (8, 8), 25)])
def test_rows_tried_or_waited_for(r, heads, chunks):
    """More than one workgroup per CU, on both sides of the chunk counts from which the rows are not tried unannounced."""
    compare_steps(r, heads, chunks * 1024 - 3, 1024, "staircase")


@pytest.mark.parametrize("r,heads,L", [(128, (5, 1), 20011), (256, (8, 1), 9000), (64, (1, 1), 40000), (32, (2, 1), 8449)])
@pytest.mark.parametrize("kind", ["one_near", "one_far", "staircase", "two_values"])
def test_threshold_found_by_the_attention_launch(r, heads, L, kind):
    """The step without waits inside a kernel: the scoring launch's rows, read by the attention launch."""
    compare_steps(r, heads, L, 1024, kind, waits=False)


def compare_steps(r, heads, L, chunk, kind, waits=True):
    import torch
    from paper_2506_02572_amd import hata
    (Hq, Hkv), B = heads, 3
    G, W = Hq // Hkv, r // 32
    print(f"[step selection] r={r} heads={heads} L={L} chunk={chunk} {kind}", flush=True)
    rng = np.random.default_rng(L + r)
    seq = np.array([L, L - chunk // 2 - 1, min(L, 2 * chunk)], np.int32)
    k_max = max(8, L // 40)
    k = np.array([k_max, 7, max(1, k_max // 3)], np.int32)
    K, V = (synth.round_to_bf16_bits(rng.standard_normal((B, Hkv, L, 128))) for _ in range(2))
    q = synth.round_to_bf16_bits(np.repeat(rng.standard_normal((B, Hkv, 1, 128)), G, 2).reshape(B, Hq, 128))
    WH = rng.standard_normal((Hkv, 128, r)).astype(np.float32)
    qcodes, _ = O.encode_query_batch(q, WH)
    # a key's code: the (shared) query code with as many bits flipped as its chunk says
    part = np.arange(L) // chunk
    last = max(1, (L - 1) // chunk)
    flips = {"one_near": np.where(part == last, 1, r - 2), "one_far": np.where(part == 0, r - 1, r // 8),
             "staircase": part * (r - 2) // last, "two_values": np.where(rng.random(L) < 0.02, 1, r - 1)}[kind]
    flips = np.clip(flips + rng.integers(0, 2, L), 0, r)
    order = np.argsort(rng.random((L, r)), axis=1)
    bits = (np.arange(r)[None, :] < flips[:, None])[np.arange(L)[:, None], order]
    mask = np.packbits(bits.reshape(L, W, 32), axis=-1, bitorder="little").view(np.uint32).reshape(L, W)
    codes = qcodes.reshape(B, Hkv, G, W)[:, :, :1, :] ^ mask[None, None]
    ref = O.decode_step(q, K, V, WH, codes.copy(), seq, k, k_max, 1 / math.sqrt(128), append=False)
    ctx = hata.Context(B, Hq, Hkv, 128, r, L, k_max, chunk=chunk, shared_device=not waits)
    if waits:
        assert ctx.hata_step_plan(B)[:2] == (1, chunk)
    else:
        assert ctx.hata_step_plan(B)[0] == 3
    out = torch.zeros((B, Hq, 128), dtype=torch.int16, device="cuda")
    out32 = torch.zeros((B, Hq, 128), dtype=torch.float32, device="cuda")
    Kd, Vd, Wd, cd, qd, sd, kd = (H.to_dev(x) for x in (K, V, WH, codes, q, seq, k))
    for turn in range(3):  # (the words of earlier launches are in the workspace)
        for n in ((1, 3, 2), (3, 1, 3))[turn % 2]:
            ctx.hata_decode_step(qd, Kd, Vd, Wd, cd, sd, kd, n, False, 1 / math.sqrt(128), out, out32)
        ctx.hata_check()
        idx = H.to_host(ctx.hata_step_buffers()[2])
        n = (2, 3)[turn % 2]
        assert np.array_equal(idx[:n], ref["idx"][:n])
        H.check_attention(H.to_host(out32)[:n], H.to_host(out, np.uint16)[:n], ref["out"][:n], kind)
    ctx.close()
