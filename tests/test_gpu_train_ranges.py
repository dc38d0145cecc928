"""The trainer at the edges of its launch rules, against the fp64 oracle: the number of 128-triplet blocks up to
which every workgroup of the gradient launch sums its query's column sums itself, and label lists whose
scores fall into one bin, spread over hundreds of octaves, or tie."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hash_train_oracle as T
from paper_2506_02572_amd import synth, train
from tests import harness as H
from tests.test_gpu_train import GRAD_TOL, make_problem


@pytest.mark.parametrize("blocks,r", [(512, 32), (513, 32), (513, 128)])
def test_step_on_both_sides_of_the_column_sum_rule(blocks, r):
    import torch
    n, n_q = blocks * train.BLOCK - 5, 3
    print(f"[train] blocks={blocks} r={r}", flush=True)
    Qb, Kb, Q, K, s, W = make_problem(n, r, seed=17)
    names = (np.arange(blocks) * 7 % n_q).astype(np.int32)
    hp = train.default_hparams(n)
    hp.lr = 0.0
    kw = dict(sigma=hp.sigma, eps=hp.eps, eta=hp.eta, lam=hp.lam, scale_sim=hp.scale_sim, scale_bal=hp.scale_bal,
              group=np.repeat(names, train.BLOCK)[:n])
    terms = T.loss_terms(Q, K, s, W, **kw)
    _, g_ref = T.loss_and_grad(Q, K, s, W, **kw)
    ctx = train.TrainContext(128, r, n)
    Wd = H.to_dev(W.copy())
    gd, ld = torch.empty_like(Wd), torch.empty(3, dtype=torch.float32, device="cuda")
    ctx.hata_train_step(H.to_dev(Qb), H.to_dev(Kb), H.to_dev(s), n, Wd, torch.zeros_like(Wd), hp, gd, ld,
                        block_query=H.to_dev(names), n_queries=n_q)
    torch.cuda.synchronize()
    assert np.max(np.abs(H.to_host(gd) - g_ref)) <= GRAD_TOL * np.max(np.abs(g_ref))
    np.testing.assert_allclose(H.to_host(ld), terms, rtol=2e-5)
    ctx.close()


@pytest.mark.parametrize("r", [32, 64, 256])
@pytest.mark.parametrize("runs", [(1,), (33, 31), (64, 1, 447), (1,) * 17, (1,) * 32, (1,) * 33, (1, 9) * 30, (1,) * 600, (600,), (70, 33, 1, 1, 1095)])
def test_step_on_runs_of_blocks(r, runs):
    """The update looks at 32 blocks at a time: all one query's, a few queries', a query each; any number of such pieces."""
    import torch
    blocks, n_q = sum(runs), len(runs)
    n = blocks * train.BLOCK - 3
    print(f"[train] runs={runs if n_q < 9 else n_q} r={r}", flush=True)
    Qb, Kb, Q, K, s, W = make_problem(n, r, seed=blocks)
    names = np.repeat(np.arange(n_q, dtype=np.int32), runs)
    hp = train.default_hparams(n)
    hp.lr = 0.0
    kw = dict(sigma=hp.sigma, eps=hp.eps, eta=hp.eta, lam=hp.lam, scale_sim=hp.scale_sim, scale_bal=hp.scale_bal,
              group=np.repeat(names, train.BLOCK)[:n])
    terms = T.loss_terms(Q, K, s, W, **kw)
    _, g_ref = T.loss_and_grad(Q, K, s, W, **kw)
    ctx = train.TrainContext(128, r, n)
    Wd = H.to_dev(W.copy())
    gd, ld = torch.empty_like(Wd), torch.empty(3, dtype=torch.float32, device="cuda")
    ctx.hata_train_step(H.to_dev(Qb), H.to_dev(Kb), H.to_dev(s), n, Wd, torch.zeros_like(Wd), hp, gd, ld,
                        block_query=H.to_dev(names), n_queries=n_q)
    torch.cuda.synchronize()
    assert np.max(np.abs(H.to_host(gd) - g_ref)) <= GRAD_TOL * np.max(np.abs(g_ref))
    np.testing.assert_allclose(H.to_host(ld), terms, rtol=2e-5)
    ctx.close()


@pytest.mark.parametrize("m", [256, 257, 20000])
@pytest.mark.parametrize("kind", ["equal", "one_bin", "octaves", "negative"])
def test_labels_of_awkward_scores(kind, m):
    import torch
    print(f"[labels] {kind} m={m}", flush=True)
    rng = np.random.default_rng(m)
    # one channel carries the score, exactly: K[i, 0] * 1
    col = {"equal": np.full(m, 3.0), "one_bin": 1.0 + rng.integers(0, 4, m) / 64.0,
           "octaves": rng.choice([-1.0, 0.0, 1.0], m) * 2.0 ** rng.integers(-90, 90, m),
           "negative": -rng.integers(1, 128, m).astype(np.float64)}[kind]
    K, q = np.zeros((m, 128), np.float32), np.zeros(128, np.float32)
    K[:, 0], q[0] = col, 1.0
    want = T.make_labels(col).astype(np.float32)
    ctx = train.TrainContext(128, 32, m)
    s = torch.empty(m, dtype=torch.float32, device="cuda")
    Kd, qd = H.to_dev(synth.round_to_bf16_bits(K)), H.to_dev(synth.round_to_bf16_bits(q))
    for _ in range(2):  # (the second call starts from what the first one left in the workspace)
        ctx.hata_train_make_labels(qd, Kd, m, s)
        torch.cuda.synchronize()
        assert np.array_equal(H.to_host(s), want)
    ctx.close()


def labels_problem(m, seed):
    rng = np.random.default_rng(seed)
    K, q = np.zeros((m, 128), np.float32), np.zeros(128, np.float32)
    K[:, 0], q[0] = rng.integers(-100, 100, m), 1.0
    return H.to_dev(synth.round_to_bf16_bits(q)), H.to_dev(synth.round_to_bf16_bits(K)), T.make_labels(K[:, 0].astype(np.float64)).astype(np.float32)


def test_labels_of_a_context_made_behind_pending_work():
    """The workspace's memory is still being written on the stream that the context is made and used on."""
    import ctypes
    import torch
    m = 5000
    q, K, want = labels_problem(m, 1)
    n = ctypes.c_size_t(0)
    train._lib().hata_train_workspace_bytes(ctypes.byref(train.hata_train_config(128, 32, m)), ctypes.byref(n))
    s = torch.empty(m, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        earlier = torch.empty(n.value + 256, dtype=torch.uint8, device="cuda")
        address = earlier.data_ptr()
        torch.cuda._sleep(20_000_000)  # some milliseconds
        earlier.fill_(1)
        del earlier
        ctx = train.TrainContext(128, 32, m)
        assert ctx.workspace.data_ptr() == address
        ctx.hata_train_make_labels(q, K, m, s)
    torch.cuda.synchronize()
    assert np.array_equal(H.to_host(s), want)
    ctx.close()


def test_first_label_call_recorded_into_a_graph():
    import torch
    m = 3000
    q, K, want = labels_problem(m, 2)
    ctx = train.TrainContext(128, 32, m)
    ctx.workspace.fill_(255)
    s = torch.zeros(m, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.hata_train_make_labels(q, K, m, s)
    torch.cuda.synchronize()
    for turn in range(4):
        print(f"[labels] graph, turn {turn}", flush=True)
        s.zero_()
        ctx.hata_train_make_labels(q, K, m, s)  # (the first one comes before any replay)
        torch.cuda.synchronize()
        assert np.array_equal(H.to_host(s), want)
        s.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(H.to_host(s), want)
    ctx.close()
