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
    (2, 130, 256, 4, 64, 1, 2, True),     # one tile of rows
    (4, 16, 448, 7, 128, 2, 7, False),    # heads of 128,
    (4, 7, 1088, 17, 128, 0, 17, True),   # two groups of waves
    (2, 25, 1088, 17, 128, 3, 16, True),
    (3, 13, 2112, 3, 64, 0, 3, False),    # several groups of heads
    (2, 20, 2048, 4, 64, 0, 4, True),
    (1, 22, 3008, 47, 128, 0, 47, False),
]
# near the line, faster by rows: one tile of rows, heads of 128 on short causal walks
BY_ROWS = [(2, 60, 256, 4, 64, 1, 2, True), (4, 9, 832, 13, 128, 0, 13, True)]


@pytest.mark.parametrize("B,Z,L,N,A,rb,re,causal", CASES + BY_ROWS)
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


@pytest.mark.parametrize("B,Z,L,N,A,rb,re,causal", [CASES[0], CASES[3], CASES[5], CASES[7], CASES[8], CASES[10]])
@pytest.mark.parametrize("std", [1.0, 4.0])
def test_backward_by_keys_is_as_exact_as_by_rows(B, Z, L, N, A, rb, re, causal, std):
    """RMS error against 64 bits, beside that of the same heads taken one at a time, which go by rows: both round P and dS once and
    the results once, from fp32 sums in other orders, so that other elements fall to either side: 2 % of the error of an
    element (2e-3 of the RMS) over 10^5 of them and more."""
    cfg = inputs.RSAConfig("k", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=rb, rank_end=re, seed=79)
    x = inputs.make_inputs(cfg)
    Q, K, V, dO = (upload(x[k], "bf16") for k in ("Q", "K", "V", "dO"))
    Q, K = Q * std, K * std       # (scores of 60: P from a rounded LSE)
    kw = dict(causal=causal, rank_begin=rb, rank_end=re, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(rsa.make_desc(K, N, **kw), Q, K, V)
    got = rsa.backward(rsa.make_desc(K, N, **kw), dO, Q, K, V, O, LSE)
    some = sorted({0, 1, B * Z // 2, B * Z - 1})
    head = lambda t, h: t.view(1, B * Z, *t.shape[2:])[:, h:h + 1].contiguous()
    err = torch.zeros(2, 3, 2, dtype=torch.float64)
    for h in some:
        q, k, v, g, o, lse = (head(t, h) for t in (Q, K, V, dO, O, LSE))
        rows = rsa.backward(rsa.make_desc(k, N, **kw), g, q, k, v, o, lse)
        ref = gradients(cfg, q, k, v, g, o)
        for i in range(3):
            for side, t in enumerate((head(got[i], h), rows[i])):
                err[side, i] += torch.stack(((t.double() - ref[i]).square().sum(), ref[i].square().sum())).cpu()
    rel = (err[..., 0] / err[..., 1]).sqrt()
    print(f"by keys {rel[0].tolist()}, by rows {rel[1].tolist()}")
    assert (rel[0] <= 1.02 * rel[1]).all()


def gradients(cfg, Q, K, V, dO, O):
    """dQ, dK, dV in 64 bits; D from the stored O that both sides are given."""
    Q, K, V, dO, O = (t.double() for t in (Q, K, V, dO, O))
    s = cfg.A ** -0.5
    S = Q @ K.mT.contiguous() * s
    if cfg.causal:
        q = torch.arange(cfg.Lq, device=Q.device) + cfg.ranks[0] * cfg.c
        S.masked_fill_(torch.arange(cfg.L, device=Q.device) > q[:, None], float("-inf"))
    P = torch.softmax(S, -1)
    dS = P * (dO @ V.mT.contiguous() - (dO * O).sum(-1, keepdim=True))
    return dS @ K * s, dS.mT.contiguous() @ Q * s, P.mT.contiguous() @ dO


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
