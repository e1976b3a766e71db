"""Several wavefronts on one partition: their states folded head by head, into a record for the merge pass or into the output.

Blocks of eight (one launch), of four and of two wavefronts, one to eight query heads per kv head (so that a wavefront has no
head, one, or several), pairs of 64-channel heads, with and without a learned rotation; lengths that leave wavefronts of a
block without a batch.  Against the oracle, with the tolerance of the decode and append tests."""
import pytest
import torch

import test_gpu_append as TA
import test_gpu_decode as TD
from paper_2604_19157_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def saw():
    from paper_2604_19157_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("G,d,dense", [(1, 128, None), (2, 128, 3), (4, 128, None), (4, 128, 4), (8, 128, None), (8, 128, 5),
                                       (1, 64, None), (2, 64, None), (4, 64, None)])
def test_block_end(saw, G, d, dense):
    def w(lens, **kw):
        return synth.make_workload("highconc", batch=len(lens), seq_lens=lens, n_q_heads=2 * G, n_kv_heads=2, head_dim=d, had_block=64,
                                   dense_seed=dense, **kw)
    TA._case(saw, w([0, 1, 64, 65, 300, 511]))                                          # eight, fused append, one launch
    TD._decode_case(saw, w([1, 0, 700, 4000, 4200]), num_splits=1, end_to_end=False)    # four on one partition
    TD._decode_case(saw, w([0, 9000, 5000]), end_to_end=False, out_dtype=torch.float16)  # cut by the lengths, four a slot
    TA._case(saw, w([3000 - 61 * k for k in range(40)] + [0]))                          # ... or two
