"""Training steps whose workgroups go through several pairs of blocks, and some just below: runs that end with the workgroup and with the
number of stages kept; another query vector in a run's later tiles and in the padding; against the fp64 oracle.  (Queries that end inside
runs and vectors that change there are in test_gpu_train_broken_runs.py.)"""
import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_train_blocks import test_step_on_blocks_of_one_query as step_on_blocks


# (blocks of 128 keys; 256 workgroups of 32 columns are a round: r = 256 has two pairs a workgroup of one query from 65 blocks, six from 258.
# Three queries of 23 blocks and nine of 8 have a pair a workgroup)
@pytest.mark.parametrize("r,keys,n_q,stray", [
    (256, 8320, 1, None), (256, 8400, 1, 300), (256, 8400, 1, 8440),  # 65 and 66 blocks; a stray row in the second stage, in the padding
    (256, 2900, 3, None), (256, 2900, 3, 2950),                       # queries of 23 blocks, which share pairs
    (256, 1024, 9, None), (64, 66000, 1, 33000),                      # queries of whole runs; three stages
    (256, 38400, 1, None), (256, 38400, 1, 1100), (256, 19200, 2, None),  # two runs of three stages; a stray row in the second run
])
def test_step_on_runs_of_pairs(r, keys, n_q, stray):
    step_on_blocks(r, keys, n_q, stray)
