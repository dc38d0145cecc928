"""Training steps whose workgroups go through runs of pairs of blocks, with queries that change inside a pair, inside a run and at a run's
end, and with query vectors that change under one name; the gradient without the uncorrelation term against the fp64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hash_train_oracle as T
from paper_2506_02572_amd import synth, train
from tests import harness as H


def form(r, blocks, queries):
    """The gradient launch's rule (hata_train_step): pairs of blocks a workgroup goes through, pairs of a run; (1, 1): no runs."""
    pairs = (blocks + 1) // 2
    pairs_32 = pairs * (r // 32)
    if pairs_32 <= 256 or blocks < 8 * queries:
        return 1, 1
    if r > 32 and pairs_32 <= 512 and queries > (4 if pairs_32 > 504 else 1):
        return 1, 1
    least = -(-pairs_32 // 256)
    runs = -(-least // 4)
    length = -(-least // runs)
    return runs * length, length


def broken(lengths, run_len):
    """Runs that hold more than one query."""
    names = np.repeat(np.arange(len(lengths)), lengths)
    return sum(len(set(names[b:b + 2 * run_len])) > 1 for b in range(0, len(names), 2 * run_len))


def gradient_and_bound(Q, K, s, W, hp, group):
    """The oracle's gradient, and what each element's terms add up to with a difference of 2 in every similarity (an error of h is absolute)."""
    kw = dict(sigma=hp.sigma, eps=hp.eps, eta=hp.eta, lam=hp.lam, scale_sim=hp.scale_sim, scale_bal=hp.scale_bal, group=group)
    _, grad = T.loss_and_grad(Q, K, s, W, **kw)
    eq, ek = (1.0 - T.relaxed_hash(X, W, hp.sigma) ** 2 for X in (Q, K))
    sim = 2.0 * hp.eps * hp.scale_sim * np.abs(s)[:, None]
    col = np.zeros((int(group.max()) + 1, W.shape[1]))
    np.add.at(col, group, np.abs(T.relaxed_hash(K, W, hp.sigma)))
    bal = 2.0 * hp.eta * hp.scale_bal * col[group]
    return grad, T.loss_terms(Q, K, s, W, **kw), hp.sigma * (np.abs(Q).T @ (sim * eq) + np.abs(K).T @ ((sim + bal / 2) * ek))


def step(r, lengths, named=True, change=(), loose=0, queries=None):
    """lengths: blocks of each query.  change: rows from which on the query vector is another, up to the next such row or query.  named
    False: block_query is NULL, and the vectors alone follow `lengths`.  loose: zero rows of the last block, past n."""
    import torch
    blocks = sum(lengths)
    n = blocks * train.BLOCK - loose
    rng = np.random.default_rng(blocks + r)
    starts = sorted(set(int(x) * train.BLOCK for x in np.cumsum([0] + list(lengths[:-1]))) | set(change))
    which = np.searchsorted(starts, np.arange(n), side="right") - 1
    # (keys off centre: the column sums do not cancel)
    Kb = synth.round_to_bf16_bits((rng.standard_normal((n, 128)) + rng.standard_normal(128)).astype(np.float32))
    Qb = synth.round_to_bf16_bits(rng.standard_normal((len(starts), 128)).astype(np.float32))[which]
    s = np.where(rng.random(n) < 0.1, 20.0 * rng.random(n), -1.0).astype(np.float32)
    W = (rng.standard_normal((128, r)) * 128 ** -0.5).astype(np.float32)
    names = np.repeat(np.arange(len(lengths), dtype=np.int32), lengths) if named else np.zeros(blocks, np.int32)
    n_q = int(names.max()) + 1
    hp = train.default_hparams(n)
    hp.lr = hp.lam = 0.0
    hp.scale_bal = hp.eps * hp.scale_sim / hp.eta * n_q / n
    Q, K = (synth.bf16_to_f32(x).astype(np.float64) for x in (Qb, Kb))
    g_ref, terms, bound = gradient_and_bound(Q, K, s, W, hp, np.repeat(names, train.BLOCK)[:n])
    ctx = train.TrainContext(128, r, n)
    Wd = H.to_dev(W.copy())
    gd, ld = torch.empty_like(Wd), torch.empty(3, dtype=torch.float32, device="cuda")
    kw = dict(block_query=H.to_dev(names), n_queries=n_q) if named else {}
    ctx.hata_train_step(H.to_dev(Qb), H.to_dev(Kb), H.to_dev(s), n, Wd, torch.zeros_like(Wd), hp, gd, ld, **kw)
    torch.cuda.synchronize()
    err = np.max(np.abs(H.to_host(gd) - g_ref) / bound)
    print(f"  error {err * 2**21:.3f} of 2^-21 of the terms; loss {H.to_host(ld)}", flush=True)
    # Some 64 roundings to 24 bits on the way of a sum -- a tile's products, the tiles and waves of a run, the runs -- of either sign: eight
    # of them.  (A lost tile of 32 rows of 123000 is 2^-13 of the terms or more.)
    assert err <= 2.0 ** -21
    np.testing.assert_allclose(H.to_host(ld)[:2], terms[:2], rtol=2e-5)
    ctx.close()


def split(kind, blocks):
    """Blocks of each query."""
    if kind == "one": return [blocks + 1]
    if kind == "two": return [blocks // 2 - 3, blocks - blocks // 2 + 3]
    if kind == "quarters": return [blocks // 4] * 4
    if kind == "four": return [1, blocks // 3, 7, blocks - blocks // 3 - 8]
    if kind == "uneven": return [1, blocks // 3, 2, blocks // 4 + 1, 5, blocks - blocks // 3 - blocks // 4 - 9]
    if kind == "mixed": return [11, 1, 1, 4, 3, 8, 16, 2, 2, 31, blocks - 79]
    return [int(kind[2:])] * -(-blocks // int(kind[2:]))


@pytest.mark.parametrize("r", [32, 64, 128, 256])
@pytest.mark.parametrize("kind", ["one", "two", "uneven", "mixed", "by150", "by23", "by9", "by7"])
def test_queries_that_end_anywhere(r, kind):
    """Batches of two and a half rounds of workgroups and more, at r = 32 of one and a half."""
    lengths = split(kind, 768 if r == 32 else 1280 * 32 // r)
    stages, run_len = form(r, sum(lengths), len(lengths))
    print(f"[train] r={r} {kind}: {sum(lengths)} blocks, {stages} pairs a workgroup, runs of {run_len}, {broken(lengths, run_len)} broken", flush=True)
    if kind != "by7":  # (a pair a workgroup)
        assert run_len >= 2 and (broken(lengths, run_len) > 0 or kind in ("one", "by150"))
    step(r, lengths, loose=37)


@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("kind,short,runs", [("one", 1, True), ("two", 0, True), ("quarters", 0, True), ("four", 0, True), ("uneven", 0, False), ("four", 1, False), ("four", 2, False), ("one", 3, True)])
def test_two_rounds(r, kind, short, runs):
    """Two rounds of workgroups, and a sixteenth, a quarter and almost a half of the pairs less."""
    pairs = 512 // (r // 32)
    blocks = 2 * (pairs - (0, pairs // 16, pairs // 4, pairs // 2 - 1)[short])
    lengths = split(kind, blocks - (kind == "one"))
    stages, run_len = form(r, sum(lengths), len(lengths))
    print(f"[train] r={r} {kind}: {sum(lengths)} blocks, {stages} pairs a workgroup, {broken(lengths, 2)} of two broken", flush=True)
    assert (run_len == 2) == runs
    step(r, lengths, loose=5)


def rows_of(pair, *rows):
    return [pair * 256 + x for x in rows]


@pytest.mark.parametrize("r,blocks", [(256, 272), (128, 520), (128, 960), (64, 1030), (32, 1030)])
@pytest.mark.parametrize("kind", ["blocks", "pairs", "some_tiles", "last_tile", "inside", "rows"])
def test_vectors_that_change_under_one_name(r, blocks, kind):
    """Every tile of one vector, another one in the run's next tile, in some waves only; rows inside a tile, in a run's first and last
    pair; every row another."""
    stages, run_len = form(r, blocks, 1)
    print(f"[train] r={r} blocks={blocks} {kind}: {stages} pairs a workgroup, runs of {run_len}", flush=True)
    assert run_len >= 2
    pairs = blocks // 2
    change = {"blocks": range(0, blocks * 128, 128), "pairs": range(0, blocks * 128, 256),
              "some_tiles": [x for p in range(pairs) if p % 3 for x in rows_of(p, 32 * (p % 5), 32 * (p % 5) + 32 * (1 + p % 3))],
              "last_tile": [x for p in range(run_len - 1, pairs, run_len) for x in rows_of(p, 224)],
              "inside": [x for p in range(pairs) if p % 2 for x in rows_of(p, 7 + 13 * (p % 17), 8 + 13 * (p % 17))],
              "rows": range(blocks * 128 - 5)}[kind]
    step(r, [blocks], named=False, change=change, loose=5)
