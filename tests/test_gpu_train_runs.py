"""Training steps whose workgroups go through several pairs of blocks: runs of one query that end with the workgroup, with the
number of stages kept, with another query, inside a pair; other query vectors in a run's first, later and last tiles; against the fp64 oracle."""
import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_train_blocks import test_step_on_blocks_of_one_query as step_on_blocks


# (blocks of 128 keys; 256 workgroups of 32 columns are a round: r = 256 has two pairs a workgroup from 66 blocks, six from 258)
@pytest.mark.parametrize("r,keys,n_q,stray", [
    (256, 8320, 1, None), (256, 8400, 1, 300), (256, 8400, 1, 8440),  # 65 and 66 blocks; a stray row in the second stage, in the padding
    (256, 2900, 3, None), (256, 2900, 3, 2950),                       # queries of 23 blocks, which share pairs
    (256, 1024, 9, None), (64, 66000, 1, 33000),                      # as many runs as queries; three stages
    (256, 38400, 1, None), (256, 38400, 1, 1100), (256, 19200, 2, None),  # two runs of three stages; a stray row in the second run
])
def test_step_on_runs_of_pairs(r, keys, n_q, stray):
    step_on_blocks(r, keys, n_q, stray)
