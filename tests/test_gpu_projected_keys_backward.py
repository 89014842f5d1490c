"""The backward of attention to few projected keys: every shape of work-group and number of splits of the rows' walk,
splits that are left without rows, keys that fill a work-group in part.  (At most 9 million elements a tensor: the chain's
bound is on the largest error, and over 25 million dQ's own bf16 roundings, rms 0.0024 of the values', reach 1.01 of it.)"""
import pytest
from test_gpu_linformer import test_linformer_chain as chain

pytestmark = pytest.mark.gpu


# (B, Z, L, N, ranks, Kp, A)
@pytest.mark.parametrize("B,Z,L,N,ranks,Kp,A", [
    (1, 12, 2176, 17, (0, 17), 64, 64),     # one block of keys per work-group, four groups, 8 splits of 34 tiles
    (1, 5, 13824, 27, (0, 27), 64, 64),     # 16 splits or more
    (1, 12, 2048, 1, (0, 1), 512, 64),      # four groups, no split
    (1, 15, 7488, 1, (0, 1), 512, 64),      # four blocks of keys, 4 splits
    (2, 20, 3136, 1, (0, 1), 64, 64),       # two blocks, two groups, 8 splits of 49 tiles, the last one with none
    (1, 3, 1088, 1, (0, 1), 320, 64),       # ragged blocks and stages
    (1, 12, 2048, 2, (0, 2), 128, 128),     # heads of 128: two blocks, two groups, 8 splits
    (2, 30, 2048, 8, (0, 8), 192, 128),
])
def test_few_keys(B, Z, L, N, ranks, Kp, A):
    chain(B, Z, L, N, ranks, Kp, A)
