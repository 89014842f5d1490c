"""The two-pass bf16 backward by keys (dK, dV while the scores are in registers, dQ from the strip of dS^T): at the lines of
its rule, with ragged key blocks and odd numbers of row tiles, one rank's share, in one group of heads and several, for each
number of groups of waves."""
import pytest
import torch

from helpers import compare_heads, gpu_forward_backward, upload
from paper_2105_13120_amd import inputs, rsa

pytestmark = pytest.mark.gpu

# (B, Z, L, N, A, first rank, last rank + 1, causal)
CASES = [
    (4, 8, 512, 4, 64, 0, 4, False),      # as few work-groups as it takes,
    (5, 16, 320, 5, 64, 0, 5, False),     # the last of a head half empty,
    (1, 48, 576, 9, 64, 1, 9, False),
    (2, 15, 1984, 31, 64, 0, 31, True),   # causal: one group of waves, two, four
    (5, 12, 704, 11, 64, 0, 11, True),
    (3, 4, 1600, 5, 64, 1, 5, True),
    (2, 60, 256, 4, 64, 1, 2, True),      # one tile of rows
    (4, 16, 448, 7, 128, 2, 7, False),    # heads of 128,
    (4, 9, 832, 13, 128, 0, 13, True),    # two groups of waves
    (2, 25, 1088, 17, 128, 3, 16, True),
    (3, 13, 2112, 3, 64, 0, 3, False),    # several groups of heads
    (2, 20, 2048, 4, 64, 0, 4, True),
    (1, 22, 3008, 47, 128, 0, 47, False),
]


@pytest.mark.parametrize("B,Z,L,N,A,rb,re,causal", CASES)
def test_backward_by_keys(B, Z, L, N, A, rb, re, causal):
    cfg = inputs.RSAConfig("k", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=rb, rank_end=re, seed=47)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED)
    compare_heads(cfg, x, out, sorted({0, B * Z // 2, B * Z - 1}), mode=rsa.MODE_STAGED)


@pytest.mark.parametrize("B,Z,L,N,A,rb,re,causal", [CASES[1], CASES[5], CASES[10]])
def test_backward_by_keys_over_its_inputs(B, Z, L, N, A, rb, re, causal):
    """Wherever its results lie, bit by bit the same."""
    cfg = inputs.RSAConfig("k", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=rb, rank_end=re, seed=53)
    x = inputs.make_inputs(cfg)
    t = {k: upload(x[k], "bf16") for k in ("Q", "K", "V", "dO")}
    desc = rsa.make_desc(t["K"], N, causal=causal, rank_begin=rb, rank_end=re, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(desc, t["Q"], t["K"], t["V"])
    grads = rsa.backward(desc, t["dO"], t["Q"], t["K"], t["V"], O, LSE)
    for over in (dict(dQ="Q", dK="K", dV="V"), dict(dQ="dO", dK="V", dV="K")):
        u = {k: v.clone() for k, v in t.items()}
        got = rsa.backward(desc, u["dO"], u["Q"], u["K"], u["V"], O, LSE, **{k: u[i] for k, i in over.items()})
        assert all(torch.equal(a, b) for a, b in zip(got, grads)), over


def test_backward_by_keys_whose_results_fill_the_workspace():
    """dK from the 65th row of K on: the workspace that every call is asked for holds all results and the strips of 128 rows of a
    head, not of all its rows, and the call goes by rows.  Either way errs at most 3.75e-3 of the RMS (tests/helpers.py, two-pass
    layout), so that the two differ by sqrt(2) times that."""
    heads, L, N, A = 126, 3200, 10, 64
    g = torch.Generator(device="cuda").manual_seed(71)
    Q, K, V, dO = (torch.randn((1, heads, L, A), generator=g, device="cuda").bfloat16() for _ in range(4))
    desc = rsa.make_desc(K, N, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(desc, Q, K, V)
    want = rsa.backward(desc, dO, Q, K, V, O, LSE)
    buf = torch.empty(K.numel() + 64 * A, dtype=K.dtype, device="cuda")
    K2, dK = buf[:K.numel()].view(K.shape), buf[64 * A:].view(K.shape)
    K2.copy_(K)
    for x, y in zip(rsa.backward(desc, dO, Q, K2, V, O, LSE, dK=dK), want):
        assert float((x.float() - y.float()).norm() / y.float().norm()) <= 2 ** 0.5 * 3.75e-3
