"""The two-pass bf16 forward where it keeps no strip: on either side of the line of its rule, with ragged last work-groups, one
rank's share, scores that spread wide or grow along a walk, and results that lie over inputs."""
import pytest
import torch

from helpers import compare_heads, gpu_forward_backward, upload
from paper_2105_13120_amd import inputs, rsa

pytestmark = pytest.mark.gpu

# (B, Z, L, N, A, first rank, last rank + 1, causal), whether a strip is kept
CASES = [
    ((1, 16, 512, 4, 64, 0, 4, False), True),       # 64 work-groups of 128 rows,
    ((1, 13, 576, 9, 64, 0, 9, False), False),      # 65: the last of a head half empty
    ((1, 20, 576, 9, 128, 0, 9, True), False),      # heads of 128, by their rows: 90 blocks of 128,
    ((4, 8, 512, 8, 128, 3, 7, False), True),       # 64 and 96 of one rank's share
    ((4, 8, 512, 8, 128, 2, 8, True), False),
    ((5, 14, 64, 1, 64, 0, 1, False), False),       # one tile of keys; too few keys for the results' room
    ((5, 14, 64, 1, 128, 0, 1, True), True),
    ((3, 22, 832, 13, 64, 0, 13, True), False),     # 256-row, 128-row work-groups and groups of waves
    ((2, 48, 1600, 5, 64, 0, 5, False), False),
    ((1, 6, 4096, 4, 64, 0, 4, True), False),
    ((1, 24, 8192, 16, 64, 15, 16, False), False),  # walks that the fused mode splits
    ((1, 16, 16384, 16, 64, 3, 4, False), False),
    ((1, 17, 16384, 16, 64, 15, 16, True), False),
    ((1, 96, 4096, 8, 128, 7, 8, True), False),
    ((1, 23, 640, 5, 192, 0, 5, False), True),
    ((1, 13, 576, 9, 128, 0, 9, True), True),       # 58
]


@pytest.mark.parametrize("case,strip", CASES)
def test_forward_in_one_pass(case, strip):
    B, Z, L, N, A, rb, re, causal = case
    cfg = inputs.RSAConfig("o", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=rb, rank_end=re, seed=59)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED, backward=False)
    compare_heads(cfg, x, out, sorted({0, B * Z // 2, B * Z - 1}), mode=rsa.MODE_STAGED, backward=False)


@pytest.mark.parametrize("case", [CASES[1][0], CASES[7][0], CASES[8][0], CASES[11][0]])
def test_forward_in_one_pass_over_its_inputs(case):
    """Wherever O lies, bit by bit the same: over an input, or from its 64th row on, with the workspace that is asked for."""
    B, Z, L, N, A, rb, re, causal = case
    cfg = inputs.RSAConfig("o", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=rb, rank_end=re, seed=61)
    x = inputs.make_inputs(cfg)
    t = {k: upload(x[k], "bf16") for k in ("Q", "K", "V")}
    desc = rsa.make_desc(t["K"], N, causal=causal, rank_begin=rb, rank_end=re, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(desc, t["Q"], t["K"], t["V"])
    for over in ("Q", "K", "V"):
        for rows in (0, 64):
            n = max(O.numel(), t[over].numel())
            buf = torch.empty(n + rows * A, dtype=torch.bfloat16, device="cuda")
            u = dict(t)
            u[over], out = buf[:t[over].numel()].view(t[over].shape), buf[rows * A:][:O.numel()].view(O.shape)
            u[over].copy_(t[over])
            got = rsa.forward(desc, u["Q"], u["K"], u["V"], O=out)
            assert torch.equal(got[0], O) and torch.equal(got[1], LSE), (over, rows)


@pytest.mark.parametrize("case", [CASES[1][0], CASES[2][0], CASES[9][0]])
@pytest.mark.parametrize("scores", ["unit", "wide", "rising"])
def test_forward_in_one_pass_is_as_exact_as_the_strip(case, scores):
    """RMS error against 64 bits, beside that of the same rows taken a head at a time, which keep the strip: both round a tile's
    probabilities to bf16 against its own maximum and results once, so that O errs alike (2 %: different elements fall to
    either side); LSE, one fp32 number of about ten, no more (1e-8: a sixth of its last bit)."""
    B, Z, L, N, A, rb, re, causal = case
    cfg = inputs.RSAConfig("o", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=rb, rank_end=re, seed=67)
    x = inputs.make_inputs(cfg)
    Q, K, V = (upload(x[k], "bf16") for k in ("Q", "K", "V"))
    if scores == "wide":
        Q, K = Q * 4, K * 4
    if scores == "rising":
        K = (K * torch.exp2(torch.linspace(-3, 3, L, device="cuda"))[:, None]).bfloat16()
    S = Q.double() @ K.double().mT.contiguous() / A ** 0.5
    if causal:
        S.masked_fill_(torch.ones(L, L, dtype=torch.bool, device="cuda").triu(1), -float("inf"))
    lse = torch.logsumexp(S, -1)
    ref = torch.softmax(S, -1) @ V.double()
    mk = dict(causal=causal, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(rsa.make_desc(K, N, **mk), Q, K, V)
    heads = [tuple(y[b:b + 1, z:z + 1].contiguous() for y in (Q, K, V)) for b in range(B) for z in range(Z)]
    by_head = [rsa.forward(rsa.make_desc(k, N, **mk), q, k, v) for q, k, v in heads]
    for name, got, parts, exact in (("O", O, 0, ref), ("LSE", LSE, 1, lse)):
        other = torch.cat([y[parts] for y in by_head], 1).view(got.shape)
        e, e_strip = (float((y.double() - exact).norm() / exact.norm()) for y in (got, other))
        print(f"{name} {scores}: {e:.2e}, strip {e_strip:.2e}")
        assert e <= 1.02 * e_strip + 1e-8, name


def inputs_of(case, seed):
    B, Z, L, N, A, rb, re, causal = case
    cfg = inputs.RSAConfig("o", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=rb, rank_end=re, seed=seed)
    x = inputs.make_inputs(cfg)
    return [upload(x[k], "bf16") for k in ("Q", "K", "V", "dO")], rsa.make_desc(upload(x["K"], "bf16"), N, causal=causal, mode=rsa.MODE_STAGED)


@pytest.mark.parametrize("case", [CASES[1][0], CASES[2][0], CASES[9][0]])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
def test_infinities_and_nan_reach_their_own_results_only(case, bad):
    """One element of V that is infinite or NaN: its column of O, for the rows that see it, is not finite, the rest stays as it
    was, bit by bit.  A NaN in Q: that row's results are NaN, the rest stays as it was."""
    (Q, K, V, _), desc = inputs_of(case, 83)
    causal = case[-1]
    O, LSE = rsa.forward(desc, Q, K, V)
    V2 = V.clone()
    V2[0, 1, 37, 10] = bad
    O2, LSE2 = rsa.forward(desc, Q, K, V2)
    first = 37 if causal else 0
    hit = O2[0, 1, first:, 10].float()
    assert torch.equal(LSE2, LSE)
    # (rows before 37 of its tile may meet 0 x infinity, as any product over a masked tile does)
    assert not hit.isfinite().any() and (hit.isnan().all() if bad != bad else (hit == bad).all())
    O2[0, 1, :, 10] = O[0, 1, :, 10]
    assert torch.equal(O2, O)
    Q2 = Q.clone()
    Q2[0, 2, 100] = float("nan")
    O2, LSE2 = rsa.forward(desc, Q2, K, V)
    assert O2[0, 2, 100].isnan().all() and LSE2[0, 2, 100].isnan()
    O2[0, 2, 100], LSE2[0, 2, 100] = O[0, 2, 100], LSE[0, 2, 100]
    assert torch.equal(O2, O) and torch.equal(LSE2, LSE)


@pytest.mark.parametrize("case", [CASES[1][0], CASES[2][0], CASES[8][0]])
@pytest.mark.parametrize("gone", [(0, 64), (64, 192), (0, 32)])
def test_tiles_whose_scores_are_all_minus_infinity(case, gone):
    """Keys that no row gives any weight, a whole tile of them first, between others, or half a tile: as if they were not there.
    RMS error as without them (2.4e-3 of the RMS), LSE to fp32 rounding."""
    (Q, K, V, _), desc = inputs_of(case, 89)
    A, causal = case[4], case[-1]
    Q, K = Q.clone(), K.clone()
    Q[..., 5] = Q[..., 5].abs() + 0.5
    K[:, :, gone[0]:gone[1], 5] = -float("inf")
    O, LSE = rsa.forward(desc, Q, K, V)
    S = Q.double() @ K.double().mT.contiguous() / A ** 0.5
    if causal:
        S.masked_fill_(torch.ones(S.shape[-2:], dtype=torch.bool, device="cuda").triu(1), -float("inf"))
    seen = slice(gone[1] if causal and gone[0] == 0 else 0, None)          # (rows before see no other key)
    S, O, LSE = S[:, :, seen], O[:, :, seen], LSE[:, :, seen]
    ref = torch.softmax(S, -1) @ V.double()
    assert float((O.double() - ref).norm() / ref.norm()) <= 3e-3
    assert float((LSE.double() - torch.logsumexp(S, -1)).abs().max()) <= 1e-5
