"""The two-pass kernels with groups of waves on a work-group's walk (few work-groups): walks shorter than the number of
groups, odd numbers of tiles and rows, one rank's share, on either side of the lines where the shapes change."""
import pytest

from helpers import compare_heads, gpu_forward_backward
from paper_2105_13120_amd import inputs, rsa

pytestmark = pytest.mark.gpu

# (B, Z, L, N, A, first rank, last rank + 1, causal)
CASES = [
    (1, 1, 64, 1, 64, 0, 1, False), (1, 3, 448, 7, 64, 0, 7, True), (1, 2, 192, 3, 128, 1, 2, False),   # four groups
    (5, 7, 320, 5, 64, 0, 5, False), (5, 7, 320, 5, 64, 0, 5, True), (2, 17, 576, 3, 64, 1, 3, True),   # two; four causal
    (1, 9, 320, 1, 256, 0, 1, False), (4, 25, 192, 3, 64, 0, 3, False), (4, 25, 448, 7, 64, 0, 7, True),
    (4, 32, 512, 8, 64, 0, 8, False), (5, 15, 320, 5, 64, 0, 5, True), (1, 12, 832, 13, 64, 0, 13, True),    # fp32: one pass, strip
    (7, 17, 448, 7, 64, 2, 7, True), (1, 11, 704, 11, 64, 0, 11, False),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,Z,L,N,A,rb,re,causal", CASES)
def test_groups_of_waves_on_a_walk(dtype, B, Z, L, N, A, rb, re, causal):
    cfg = inputs.RSAConfig("g", B=B, Z=Z, L=L, A=A, N=N, dtype=dtype, causal=causal, rank_begin=rb, rank_end=re, seed=43)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED)
    compare_heads(cfg, x, out, sorted({0, B * Z // 2, B * Z - 1}), mode=rsa.MODE_STAGED)


# fp32 forward of four groups: as many steps of 32 keys as waves, fewer, more
STEP_CASES = [((1, 3, 128, 2, 64, 0, 2, False), True), ((1, 3, 128, 2, 64, 1, 2, True), True), ((2, 2, 64, 1, 64, 0, 1, True), True),
              ((1, 3, 192, 3, 64, 0, 3, True), False), ((1, 3, 512, 4, 64, 0, 1, True), True), ((1, 3, 384, 2, 64, 0, 1, True), False)]


@pytest.mark.parametrize("case,one_step", STEP_CASES)
def test_f32_walks_of_one_step(case, one_step):
    B, Z, L, N, A, rb, re, causal = case
    cfg = inputs.RSAConfig("s", B=B, Z=Z, L=L, A=A, N=N, dtype="f32", causal=causal, rank_begin=rb, rank_end=re, seed=73)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED, backward=False)
    compare_heads(cfg, x, out, list(range(B * Z)), mode=rsa.MODE_STAGED, backward=False)
