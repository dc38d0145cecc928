"""Training steps on blocks that hold one query vector, blocks that do not, and both side by side, against the fp64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hash_train_oracle as T
from paper_2506_02572_amd import synth, train
from tests import harness as H
from tests.test_gpu_train import GRAD_TOL


@pytest.mark.parametrize("r", [32, 64, 128, 256])
@pytest.mark.parametrize("keys,n_q,stray", [(1, 1, None), (128, 2, None), (300, 3, None), (300, 3, 290), (300, 3, 384), (900, 2, 1024),
                                            (130, 16, None), (130, 17, None), (130, 17, 4000)])
def test_step_on_blocks_of_one_query(r, keys, n_q, stray):
    """n_q queries against `keys` keys each, zero rows behind them; `stray`: a row with another query vector, which takes its
    block out of the rule (a padding row too: its label is 0, its query is not)."""
    import torch
    print(f"[train] r={r} keys={keys} queries={n_q} stray={stray}", flush=True)
    rows = -(-keys // train.BLOCK) * train.BLOCK
    n = n_q * rows
    qb = synth.train_vectors(n_q + 1, seed=7 + keys, tensor_id=synth.TID_Q)
    kb = synth.train_vectors(keys, seed=7 + keys, tensor_id=synth.TID_K)
    Qb, Kb, s = np.zeros((n_q, rows, 128), np.uint16), np.zeros((n_q, rows, 128), np.uint16), np.zeros((n_q, rows), np.float32)
    Qb[:, :keys], Kb[:, :keys] = qb[:n_q, None], kb
    for j in range(n_q):
        s[j, :keys] = T.make_labels(synth.bf16_to_f32(kb).astype(np.float64) @ synth.bf16_to_f32(qb[j]).astype(np.float64))
    Qb, Kb, s = Qb.reshape(n, 128), Kb.reshape(n, 128), s.reshape(n)
    if stray is not None:
        Qb[stray] = qb[n_q]
    Q, K = (synth.bf16_to_f32(x).astype(np.float64) for x in (Qb, Kb))
    W = synth.fill_f32(7, synth.TID_WH, (128, r), 1.0 / np.sqrt(128.0))
    names = np.repeat(np.arange(n_q, dtype=np.int32), rows // train.BLOCK)
    hp = train.default_hparams(n)
    hp.lr, hp.scale_bal = 0.0, 1.0 / (n * keys)
    kw = dict(sigma=hp.sigma, eps=hp.eps, eta=hp.eta, lam=hp.lam, scale_sim=hp.scale_sim, scale_bal=hp.scale_bal,
              group=np.repeat(names, train.BLOCK))
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
