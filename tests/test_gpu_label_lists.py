"""Labels from candidate lists of lengths around what a workgroup ranks (16), what its lanes take in one batch of loads (512) and what
one turn of the launch's workgroups covers; against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hash_train_oracle as T
from paper_2506_02572_amd import synth, train
from tests import harness as H


@pytest.mark.parametrize("m,listed", [(150, 15), (150, 16), (150, 17), (150, 96), (5000, 511), (5000, 512), (5000, 513), (5000, 1040), (5000, 4999)])
def test_labels_of_a_list_of_this_length(m, listed):
    import torch
    print(f"[labels] m={m} listed={listed}", flush=True)
    rng = np.random.default_rng(m + listed)
    # `listed` scores share the upper bin (four values of it, so that most tie), the others lie far below
    col = np.full(m, -100.0)
    col[rng.permutation(m)[:listed]] = 1.0 + rng.integers(0, 4, listed) / 64.0
    K, q = np.zeros((m, 128), np.float32), np.zeros(128, np.float32)
    K[:, 0], q[0] = col, 1.0
    ctx = train.TrainContext(128, 32, m)
    s = torch.empty(m, dtype=torch.float32, device="cuda")
    ctx.hata_train_make_labels(H.to_dev(synth.round_to_bf16_bits(q)), H.to_dev(synth.round_to_bf16_bits(K)), m, s)
    torch.cuda.synchronize()
    assert np.array_equal(H.to_host(s), T.make_labels(col).astype(np.float32))
    ctx.close()


# n_pos = 5121: four candidates a lane from here on; lists of the expected length, of one more than a whole number of turns, of every score
@pytest.mark.parametrize("m,listed", [(51210, 5120), (51210, 5121), (51210, 5185), (51209, 5185), (51210, 20000), (51210, 51210), (51209, 51209), (60000, 6000), (60007, 30001)])
def test_labels_of_a_long_list(m, listed):
    test_labels_of_a_list_of_this_length(m, listed)
