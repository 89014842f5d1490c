"""GPU parity of the staged (two-pass) kernels against the fp64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check, compare_heads, download, gpu_forward_backward, upload
from paper_2105_13120_amd import inputs, rsa

pytestmark = pytest.mark.gpu


def small_cfg(dtype, causal=False, B=2, Z=2, L=256, N=4, rb=0, re=-1, seed=3, A=64):
    return inputs.RSAConfig("t", B=B, Z=Z, L=L, A=A, N=N, dtype=dtype, causal=causal,
                            rank_begin=rb, rank_end=re, seed=seed)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("causal", [False, True])
def test_each_step_against_the_oracle(dtype, causal):
    """Every named step of one rank's ring walk, checked on its own output."""
    cfg = small_cfg(dtype, causal, rb=1, re=3)      # ranks 1 and 2 of 4; check rank n = 2
    x = inputs.make_inputs(cfg)
    n, c, L, N = 2, cfg.c, cfg.L, cfg.N
    heads = cfg.B * cfg.Z
    rows = slice((n - 1) * c, (n - 0) * c)           # rank n's rows inside Q (which starts at rank 1)
    Q, K, V, dO = (upload(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    desc = rsa.make_desc(K, N, causal=causal, rank_begin=1, rank_end=3, mode=rsa.MODE_STAGED)
    tdt = Q.dtype
    dev = Q.device
    q64 = x["Q"][:, :, rows].astype(np.float64)
    do64 = x["dO"][:, :, rows].astype(np.float64)
    k64, v64 = x["K"].astype(np.float64), x["V"].astype(np.float64)
    O_ref, LSE_ref, S_ref, P_ref = oracle.forward(q64, k64, v64, q0=n * c, causal=causal, want_scores=True)
    dQ_ref, dK_ref, dV_ref, dP_ref, dS_ref = oracle.backward(q64, k64, v64, do64, q0=n * c,
                                                            causal=causal, want_scores=True)

    # stage 1: S^n_j for every ring step
    S = torch.full((cfg.B, cfg.Z, c, L), float("nan"), dtype=torch.float32, device=dev)
    for t in range(N):
        rsa.qk_step(desc, n, (n - t) % N, Q, K, S)
    S_h = download(S)
    assert np.array_equal(np.isneginf(S_h), np.isneginf(S_ref))
    fin = np.isfinite(S_ref)
    tol = 1e-5 if dtype == "f32" else 1e-5  # inputs are exact in both; fp32 accumulate
    assert np.abs(S_h[fin] - S_ref[fin]).max() < tol * 10

    # softmax over the full row
    P = torch.empty((cfg.B, cfg.Z, c, L), dtype=tdt, device=dev)
    LSE = torch.zeros((cfg.B, cfg.Z, cfg.Lq), dtype=torch.float32, device=dev)
    rsa.row_softmax(desc, n, S, P, LSE)
    P_h = download(P)
    assert np.abs(P_h - P_ref).max() <= (1e-6 if dtype == "f32" else 2 ** -8 * P_ref.max())
    assert np.abs(download(LSE)[:, :, rows] - LSE_ref).max() < 1e-4
    assert (download(LSE)[:, :, : (n - 1) * c] == 0).all()      # other ranks' rows untouched

    # stage 2: O^n = sum_j P^n_j V^j, accumulated step by step
    Oacc = torch.empty((cfg.B, cfg.Z, c, 64), dtype=torch.float32, device=dev)
    first = True
    for t in range(N):
        j = (n - t) % N
        rsa.av_step(desc, n, j, P, V, Oacc, not first)
        first = False
    check("Oacc", download(Oacc), O_ref, dtype)
    Ost = torch.empty((cfg.B, cfg.Z, c, 64), dtype=tdt, device=dev)
    rsa.store(desc, Oacc, Ost)
    check("O", download(Ost), O_ref, dtype)

    # backward steps.  D from the oracle's O rounded to the storage dtype.
    O_full = torch.zeros_like(Q)
    O_full[:, :, rows] = torch.from_numpy(O_ref).to(tdt).cuda()
    D = torch.zeros((cfg.B, cfg.Z, cfg.Lq), dtype=torch.float32, device=dev)
    rsa.bwd_rowdot(desc, n, dO, O_full, D)
    D_ref = (do64 * download(O_full[:, :, rows])).sum(-1)
    assert np.abs(download(D)[:, :, rows] - D_ref).max() < 1e-4

    dP = torch.empty_like(S)
    for t in range(N):
        rsa.dp_step(desc, n, (n - t) % N, dO, V, dP)
    assert np.abs(download(dP) - dP_ref).max() < 1e-4

    dS = torch.empty_like(P)
    rsa.softmax_bwd(desc, n, P, dP, D, dS)
    if dtype == "f32":
        assert np.abs(download(dS) - dS_ref).max() < 1e-5
    else:
        # element by element: dS = bf16(bf16(P) (dP - D)) is two roundings of unit roundoff 2^-8
        # each, plus P times the error that the rounding of O left in D
        dD = np.abs(download(D)[:, :, rows] - (do64 * O_ref).sum(-1))[..., None]
        bound = 2.05 * 2.0 ** -8 * np.abs(dS_ref) + 1.01 * P_ref * dD + 1e-7
        assert (np.abs(download(dS) - dS_ref) <= bound).all()

    dQacc = torch.empty((cfg.B, cfg.Z, c, 64), dtype=torch.float32, device=dev)
    dKacc = torch.zeros((cfg.B, cfg.Z, L, 64), dtype=torch.float32, device=dev)
    dVacc = torch.zeros_like(dKacc)
    first = True
    for t in range(N):
        j = (n - t) % N
        rsa.dq_step(desc, n, j, dS, K, dQacc, not first)
        rsa.dk_step(desc, n, j, dS, Q, dKacc, False)     # each chunk is visited once
        rsa.dv_step(desc, n, j, P, dO, dVacc, False)
        first = False
    check("dQ", download(dQacc), dQ_ref, dtype)
    check("dK", download(dKacc), dK_ref, dtype)
    check("dV", download(dVacc), dV_ref, dtype)


def test_config_tiny_f32_forward():
    """The small fp32 workload (tiny_f32: B1 Z2 L256 N4), forward only, max abs err <= 1e-4."""
    cfg = inputs.CONFIGS["tiny_f32"]
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED, backward=False)
    errs = compare_heads(cfg, x, out, [0, 1], backward=False, mode=rsa.MODE_STAGED)
    assert errs["O"] <= 1e-4


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("causal,rb,re", [(False, 0, -1), (True, 0, -1), (False, 1, 3), (True, 2, 4)])
def test_staged_forward_backward(dtype, causal, rb, re):
    cfg = small_cfg(dtype, causal, B=1, Z=3, L=384, N=6, rb=rb, re=re, seed=11)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED)
    compare_heads(cfg, x, out, [0, 1, 2], mode=rsa.MODE_STAGED)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("A,causal,rb,re", [(128, False, 0, -1), (128, True, 1, 3), (192, True, 0, -1)])
def test_staged_heads_wider_than_64(dtype, A, causal, rb, re):
    """The two-pass layout takes any head size that is a multiple of 64 (up to 256)."""
    cfg = small_cfg(dtype, causal, B=1, Z=2, L=384, N=3, rb=rb, re=re, seed=29, A=A)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED)
    compare_heads(cfg, x, out, [0, 1], mode=rsa.MODE_STAGED)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,N,causal", [(5120, 5, False), (8192, 4, True)])
def test_staged_forward_with_long_rows(dtype, L, N, causal):
    """Rows of more than 4096 scores: the softmax keeps a row in the registers of one work-group."""
    cfg = small_cfg(dtype, causal, B=1, Z=1, L=L, N=N, rb=N - 1, re=N, seed=31)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED, backward=False)
    compare_heads(cfg, x, out, [0], backward=False, mode=rsa.MODE_STAGED)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_staged_explicit_softmax_scale(dtype):
    """rsa_desc.scale other than 1/sqrt(A) through the two-pass kernels."""
    import dataclasses
    cfg = dataclasses.replace(small_cfg(dtype, True, B=1, Z=2, L=384, N=3, seed=73), att_scale=0.2)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED)
    compare_heads(cfg, x, out, [0, 1], mode=rsa.MODE_STAGED)


@pytest.mark.parametrize("dtype,kw,heads", [
    ("f32", dict(B=1, Z=1, L=192, N=3), [0]),                          # one and a half row tiles, ragged key block
    ("bf16", dict(B=1, Z=1, L=64, N=1), [0]),                          # a single tile
    ("bf16", dict(B=1, Z=1, L=128, N=1), [0]),                         # as many tiles as are requested ahead, one more,
    ("bf16", dict(B=1, Z=2, L=192, N=3), [0, 1]),                      # and walks that start late
    ("bf16", dict(B=1, Z=2, L=448, N=7, rb=2, re=5, causal=True), [0, 1]),
    ("bf16", dict(B=1, Z=1, L=320, N=5, causal=True, A=192), [0]),
    ("bf16", dict(B=4, Z=9, L=512, N=4, causal=True), [0, 17, 35]),    # more work-groups: one tile ahead
    ("f32", dict(B=1, Z=2, L=448, N=7, rb=2, re=5, causal=True, A=256), [0, 1]),
    ("bf16", dict(B=1, Z=2, L=448, N=7, rb=2, re=5, causal=True, A=256), [0, 1]),
    ("bf16", dict(B=2, Z=15, L=2048, N=4), [0, 9, 10, 29]),            # heads in several groups
    ("f32", dict(B=1, Z=1, L=8448, N=11, causal=True), [0]),           # rows in several groups: fp32 accumulators
    ("bf16", dict(B=1, Z=1, L=12288, N=12, causal=True), [0]),
])
def test_staged_strip_groups_and_edges(dtype, kw, heads):
    """How the strips are cut: tile edges, groups of heads, groups of rows with dK, dV summed across them."""
    cfg = small_cfg(dtype, seed=83, **dict(dict(causal=False), **kw))
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED)
    compare_heads(cfg, x, out, heads, mode=rsa.MODE_STAGED)


def by_steps(cfg, Q, K, V, dO):
    """The two-pass forward and backward of cfg's ranks put together from the step-level entry points."""
    rb, re = cfg.ranks
    N, c, (B, Z, L, A) = cfg.N, cfg.c, K.shape
    desc = rsa.make_desc(K, N, causal=cfg.causal, rank_begin=rb, rank_end=re, mode=rsa.MODE_STAGED)
    f32 = lambda *s: torch.zeros(s, dtype=torch.float32, device=K.device)
    O, LSE, D, dQ = torch.empty_like(Q), f32(B, Z, cfg.Lq), f32(B, Z, cfg.Lq), torch.empty_like(Q)
    dK, dV, S, dP, acc = f32(B, Z, L, A), f32(B, Z, L, A), f32(B, Z, c, L), f32(B, Z, c, L), f32(B, Z, c, A)
    P, dS, one = torch.empty_like(S, dtype=K.dtype), torch.empty_like(S, dtype=K.dtype), torch.empty_like(acc, dtype=K.dtype)
    for n in range(rb, re):
        rows = slice((n - rb) * c, (n - rb + 1) * c)
        ring = [(n - t) % N for t in range(N)]
        for j in ring:
            rsa.qk_step(desc, n, j, Q, K, S)
        rsa.row_softmax(desc, n, S, P, LSE)
        for t, j in enumerate(ring):
            rsa.av_step(desc, n, j, P, V, acc, t > 0)
        rsa.store(desc, acc, one)
        O[:, :, rows] = one
        rsa.bwd_rowdot(desc, n, dO, O, D)
        for j in ring:
            rsa.dp_step(desc, n, j, dO, V, dP)
        rsa.softmax_bwd(desc, n, P, dP, D, dS)
        for t, j in enumerate(ring):
            rsa.dq_step(desc, n, j, dS, K, acc, t > 0)
            rsa.dk_step(desc, n, j, dS, Q, dK, True)
            rsa.dv_step(desc, n, j, P, dO, dV, True)
        rsa.store(desc, acc, one)
        dQ[:, :, rows] = one
    return dict(O=O, LSE=LSE, dQ=dQ, dK=dK, dV=dV)


def exact(cfg, Q, K, V, dO):
    """The same in 64 bits."""
    Q, K, V, dO = (t.double() for t in (Q, K, V, dO))
    s = cfg.A ** -0.5
    S = Q @ K.transpose(2, 3).contiguous() * s
    if cfg.causal:
        q = torch.arange(cfg.Lq, device=Q.device) + cfg.ranks[0] * cfg.c
        S.masked_fill_(torch.arange(cfg.L, device=Q.device) > q[:, None], float("-inf"))
    LSE = torch.logsumexp(S, -1)
    P = torch.exp(S - LSE[..., None])
    O = P @ V
    dS = P * (dO @ V.transpose(2, 3).contiguous() - (dO * O).sum(-1, keepdim=True))
    return dict(O=O, LSE=LSE, dQ=dS @ K * s, dK=dS.transpose(2, 3).contiguous() @ Q * s,
                dV=P.transpose(2, 3).contiguous() @ dO)


@pytest.mark.parametrize("kw,std", [
    (dict(L=512, N=4), 1.0),
    (dict(L=512, N=8), 4.0),                                        # scores of 60: what LSE's own rounding would cost
    (dict(L=512, N=4, A=256), 1.0),
    (dict(L=1984, N=1, A=128), 1.0),
    (dict(L=2048, N=8, rb=3, re=4, A=192, causal=True), 1.0),
    (dict(L=4096, N=8), 0.3),                                       # long sums of values of one size
    (dict(L=8448, N=11, causal=True, Z=1), 1.0),                    # rows in several groups
])
def test_f32_is_as_exact_as_its_steps(kw, std):
    """fp32 keeps the precision of the steps it fuses: the softmax by the row's own statistics, no row term inside a
    contraction, sums over keys and rows in short chains.  Error: RMS against 64 bits over RMS of the result.  Two
    fp32 pipelines that round in different places differ by a few percent of their error: at most 1.1 times the
    steps' is allowed (measured 0.23 to 0.52, LSE 0.42 to 1.01; with row terms inside the contractions, one chain per sum and P from the rounded LSE,
    2 to 6)."""
    cfg = small_cfg("f32", **dict(dict(B=1, Z=2, seed=89), **kw))
    x = inputs.make_inputs(cfg)
    Q, K, V, dO = (upload(x[k], "f32") for k in ("Q", "K", "V", "dO"))
    Q, K = Q * std, K * std
    ref, steps = exact(cfg, Q, K, V, dO), by_steps(cfg, Q, K, V, dO)
    desc = rsa.make_desc(K, cfg.N, causal=cfg.causal, rank_begin=cfg.ranks[0], rank_end=cfg.ranks[1], mode=rsa.MODE_STAGED)
    got = dict(zip(("O", "LSE"), rsa.forward(desc, Q, K, V)))
    got.update(zip(("dQ", "dK", "dV"), rsa.backward(desc, dO, Q, K, V, got["O"], got["LSE"])))
    for k, r in ref.items():
        e, e_steps = (float((t[k].double() - r).norm() / r.norm()) for t in (got, steps))
        assert e <= 1.1 * e_steps, f"{k}: {e:.2e}, by steps {e_steps:.2e}"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kw", [
    dict(B=2, Z=3, L=512, N=4, causal=True),
    dict(B=1, Z=1, L=192, N=1, A=256),                  # results larger than the strips
    dict(B=4, Z=5, L=2048, N=4),                        # heads in several groups
    dict(B=1, Z=1, L=8448, N=11),                       # rows in several groups
])
def test_staged_results_over_inputs(dtype, kw):
    """Gradients and O may be written over what they are computed from: same results as in buffers of their own (to the
    order of the sums over groups of rows)."""
    cfg = small_cfg(dtype, **dict(dict(seed=91), **kw))
    x = inputs.make_inputs(cfg)
    t = {k: upload(x[k], dtype) for k in ("Q", "K", "V", "dO")}
    desc = rsa.make_desc(t["K"], cfg.N, causal=cfg.causal, mode=rsa.MODE_STAGED)
    t["O"], t["LSE"] = rsa.forward(desc, t["Q"], t["K"], t["V"])
    grads = dict(zip(("dQ", "dK", "dV"), rsa.backward(desc, t["dO"], t["Q"], t["K"], t["V"], t["O"], t["LSE"])))
    tol = 1e-6 if dtype == "f32" else 1e-3

    def same(got, ref, what):
        assert float((got.float() - ref.float()).norm() / ref.float().norm()) <= tol, what

    for over in (dict(dQ="Q"), dict(dQ="dO"), dict(dV="dO"), dict(dK="Q"), dict(dQ="K", dV="Q"), dict(dQ="O", dK="V"),
                 dict(dQ="Q", dK="K", dV="V")):
        u = {k: v.clone() for k, v in t.items()}
        out = rsa.backward(desc, u["dO"], u["Q"], u["K"], u["V"], u["O"], u["LSE"], **{k: u[i] for k, i in over.items()})
        for (k, ref), got in zip(grads.items(), out):
            same(got, ref, (over, k))
    for i in ("Q", "K", "V"):
        u = {k: v.clone() for k, v in t.items()}
        O, LSE = rsa.forward(desc, u["Q"], u["K"], u["V"], O=u[i])
        same(O, t["O"], i)
        assert float((LSE - t["LSE"]).abs().max()) <= 1e-5
    # shifted by 64 rows: all results wait, or the workspace is too small for them
    q = t["Q"].numel()
    buf = torch.empty(q + 64 * cfg.A, dtype=t["Q"].dtype, device="cuda")
    Q, dQ = (buf[i:i + q].view(t["Q"].shape) for i in (0, 64 * cfg.A))
    Q.copy_(t["Q"])
    args = (desc, t["dO"], Q, t["K"], t["V"], t["O"], t["LSE"], dQ)
    big = torch.empty(rsa.workspace_bytes(desc, True) + 4 * q * 4, dtype=torch.uint8, device="cuda")
    with pytest.raises(rsa.RSAError) as e:
        rsa.backward(*args, ws=big[:q])
    assert e.value.status == -4
    for (k, ref), got in zip(grads.items(), rsa.backward(*args, ws=big)):
        same(got, ref, ("shifted", k))


@pytest.mark.parametrize("A,L", [(64, 256), (64, 1024), (128, 512)])     # forward in one pass; with the strip
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
def test_f32_infinities_and_nan_reach_their_own_results_only(A, L, bad):
    """One element of V or dO that is infinite or NaN: its column of O or dV becomes what 64 bits give, the rest stays
    as it was, bit by bit (the split of a number is formed beside that of its neighbour)."""
    x = inputs.make_inputs(small_cfg("f32", B=1, Z=2, L=L, N=1, A=A, seed=97))
    Q, K, V, dO = (upload(x[k], "f32") for k in ("Q", "K", "V", "dO"))
    desc = rsa.make_desc(K, 1, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(desc, Q, K, V)
    dQ, dK, dV = rsa.backward(desc, dO, Q, K, V, O, LSE)
    P = torch.softmax(Q[0, 0].double() @ K[0, 0].double().T * A ** -0.5, -1)
    for a in (10, 21):

        def check_column(got, clean, ref):
            assert torch.equal(got[0, 0, :, a].isnan(), ref.isnan())
            assert torch.equal(got[0, 0, :, a][ref.isinf()].double(), ref[ref.isinf()])
            got = got.clone()
            got[0, 0, :, a] = clean[0, 0, :, a]
            assert torch.equal(got, clean)

        V2, dO2 = V.clone(), dO.clone()
        V2[0, 0, 37, a] = dO2[0, 0, 37, a] = bad
        O2, LSE2 = rsa.forward(desc, Q, K, V2)
        check_column(O2, O, (P @ V2[0, 0, :, a:a + 1].double())[:, 0])
        assert torch.equal(LSE2, LSE)
        _, _, dV2 = rsa.backward(desc, dO2, Q, K, V, O, LSE)
        check_column(dV2, dV, (P.T @ dO2[0, 0, :, a:a + 1].double())[:, 0])


@pytest.mark.parametrize("A,L,std,causal", [(64, 512, 4.0, False), (64, 1024, 8.0, True), (128, 512, 4.0, False), (192, 512, 4.0, False),
                                            (256, 512, 4.0, True)])
def test_f32_gradients_of_scores_that_spread_wide(A, L, std, causal):
    """Where scores reach 60 and more, the gradients err by what the scores do.  One rounding of every score to fp32 is the
    measure: a score's sum is rounded after every 8 of A products, at the sizes that the partial sums have by then,
    which adds up to sqrt(A / 16) single roundings (2 to 4); as much again is allowed for what else rounds, and for
    chance where few rows count (ten seeds of each: 0.9 to 1.7 of that sum).  With the five small products of split numbers
    in the same accumulator there are six times as many roundings, 2.4 times the sum."""
    x = inputs.make_inputs(small_cfg("f32", causal, B=1, Z=2, L=L, N=1, A=A, seed=101))
    Q, K, V, dO = (upload(x[k], "f32") for k in ("Q", "K", "V", "dO"))
    Q, K = Q * std, K * std

    def gradients(of_scores):
        q, k, v, g = (t.double() for t in (Q, K, V, dO))
        S = of_scores(q @ k.transpose(2, 3).contiguous() * A ** -0.5)
        if causal:
            S = S.masked_fill(torch.ones(L, L, device="cuda").triu(1).bool(), float("-inf"))
        LSE = torch.logsumexp(S, -1)
        P = torch.exp(S - LSE[..., None])
        O = P @ v
        dS = P * (g @ v.transpose(2, 3).contiguous() - (g * O).sum(-1, keepdim=True))
        return O, LSE, dS @ k * A ** -0.5, dS.transpose(2, 3).contiguous() @ q * A ** -0.5, P.transpose(2, 3).contiguous() @ g

    ref, rounded = gradients(lambda S: S), gradients(lambda S: S.float().double())
    desc = rsa.make_desc(K, 1, causal=causal, mode=rsa.MODE_STAGED)
    got = rsa.backward(desc, dO, Q, K, V, ref[0].float(), ref[1].float())
    for name, t, r, one in zip(("dQ", "dK", "dV"), got, ref[2:], rounded[2:]):
        ratio = float((t.double() - r).norm() / (one - r).norm())
        print(f"A{A} L{L} {name}: {ratio:.2f} of one rounding of the scores")
        assert ratio <= 2 * (A / 16) ** 0.5, name


@pytest.mark.parametrize("k", [0, 100, 112, 118])
def test_f32_small_numbers(k):
    """Numbers are split to 2^-24 of themselves down to 2^-110 and to 2^-134 below: V and dO times 2^-k.  An element of O or
    dV is a sum of products with probabilities, each off by the split of either factor; the sums' own roundings, in chains
    of 32 and two dozen in all, are 2^-21 of the magnitudes at most.  Subnormal results have 2^-149."""
    x = inputs.make_inputs(small_cfg("f32", B=1, Z=2, L=512, N=1, seed=103))
    Q, K, V, dO = (upload(x[i], "f32") for i in ("Q", "K", "V", "dO"))
    V, dO = V * 2.0 ** -k, dO * 2.0 ** -k
    desc = rsa.make_desc(K, 1, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(desc, Q, K, V)
    _, _, dV = rsa.backward(desc, dO, Q, K, V, O, LSE)
    P = torch.softmax(Q.double() @ K.double().transpose(2, 3).contiguous() * 64 ** -0.5, -1)
    for got, p, y in ((O, P, V.double()), (dV, P.transpose(2, 3).contiguous(), dO.double())):
        ref, size = p @ y, p @ y.abs()
        bound = 2.0 ** -21 * size + 2.0 ** -134 * p.sum(-1, keepdim=True) + 2.0 ** -149
        assert bool(((got.double() - ref).abs() <= bound).all())
        if k <= 100:
            assert float((got.double() - ref).norm() / ref.norm()) <= 4e-7


@pytest.mark.parametrize("dtype,kw", [
    ("f32", dict(B=4, Z=8, L=2048, N=8)),                 # forward in one pass,
    ("f32", dict(B=16, Z=12, L=512, N=4, causal=True)),   # O over K and V a few heads at a time
    ("f32", dict(B=1, Z=3, L=320, N=5)),                  # groups of waves on a walk
    ("f32", dict(B=2, Z=12, L=1984, N=1, causal=True)),   # strips, in groups of heads
    ("f32", dict(B=1, Z=9, L=2048, N=4, A=128)),
    ("bf16", dict(B=2, Z=16, L=2048, N=4)),
    ("bf16", dict(B=1, Z=24, L=2048, N=4, A=128, causal=True)),
])
def test_staged_results_over_inputs_round_alike(dtype, kw):
    """The kernels and their shapes are chosen by the call, not by how many heads' results wait in the workspace at a time:
    bit-identical wherever the results lie (all rows of a head fit a group here)."""
    cfg = small_cfg(dtype, **dict(dict(seed=107), **kw))
    x = inputs.make_inputs(cfg)
    t = {k: upload(x[k], dtype) for k in ("Q", "K", "V", "dO")}
    desc = rsa.make_desc(t["K"], cfg.N, causal=cfg.causal, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(desc, t["Q"], t["K"], t["V"])
    for i in ("Q", "K", "V"):
        u = {k: v.clone() for k, v in t.items()}
        got = rsa.forward(desc, u["Q"], u["K"], u["V"], O=u[i])
        assert torch.equal(got[0], O) and torch.equal(got[1], LSE), i
    grads = rsa.backward(desc, t["dO"], t["Q"], t["K"], t["V"], O, LSE)
    u = {k: v.clone() for k, v in t.items()}
    got = rsa.backward(desc, u["dO"], u["Q"], u["K"], u["V"], O, LSE, dQ=u["Q"], dK=u["K"], dV=u["V"])
    for a, b in zip(got, grads):
        assert torch.equal(a, b)


@pytest.mark.parametrize("kw", [dict(B=4, Z=8, L=2048, N=8), dict(B=16, Z=12, L=512, N=4, causal=True), dict(B=1, Z=3, L=320, N=5)])
@pytest.mark.parametrize("over", ["Q", "K", "V"])
def test_f32_forward_over_shifted_inputs(kw, over):
    """O from the 64th row of an input on, in one pass, with the workspace that the descriptor asks for."""
    cfg = small_cfg("f32", **dict(dict(seed=109), **kw))
    x = inputs.make_inputs(cfg)
    t = {k: upload(x[k], "f32") for k in ("Q", "K", "V")}
    desc = rsa.make_desc(t["K"], cfg.N, causal=cfg.causal, mode=rsa.MODE_STAGED)
    O, LSE = rsa.forward(desc, t["Q"], t["K"], t["V"])
    n = O.numel()
    buf = torch.empty(n + 64 * 64, device="cuda")
    u = dict(t)
    u[over], out = buf[:n].view(O.shape), buf[64 * 64:].view(O.shape)
    u[over].copy_(t[over])
    got = rsa.forward(desc, u["Q"], u["K"], u["V"], O=out)
    assert torch.equal(got[0], O) and torch.equal(got[1], LSE)


@pytest.mark.parametrize("B,Z,L,N,causal,on_a_walk", [
    (4, 8, 2048, 8, False, 1), (1, 35, 1536, 1, True, 1), (3, 8, 1536, 6, True, 2), (1, 12, 1024, 4, True, 4),
])
@pytest.mark.parametrize("scores", ["unit", "wide", "rising"])
def test_f32_one_pass_on_long_walks(B, Z, L, N, causal, on_a_walk, scores):
    """The fp32 forward in one pass where walks are longer than 512 keys: as exact as its steps, also where scores reach 60,
    and where they grow along the keys, so that every step of a walk moves the reference that a row's sums are kept to."""
    cfg = small_cfg("f32", causal, B=B, Z=Z, L=L, N=N, seed=113)
    x = inputs.make_inputs(cfg)
    Q, K, V, dO = (upload(x[k], "f32") for k in ("Q", "K", "V", "dO"))
    if scores == "wide":
        Q, K = Q * 4, K * 4
    if scores == "rising":  # keys from an eighth to eight times their length
        K = K * torch.exp2(torch.linspace(-3, 3, L, device="cuda"))[:, None]
    ref, steps = exact(cfg, Q, K, V, dO), by_steps(cfg, Q, K, V, dO)
    O, LSE = rsa.forward(rsa.make_desc(K, N, causal=causal, mode=rsa.MODE_STAGED), Q, K, V)
    for k, t in (("O", O), ("LSE", LSE)):
        e, e_steps = (float((y.double() - ref[k]).norm() / ref[k].norm()) for y in (t, steps[k]))
        print(f"{k} {scores}: {e:.2e}, by steps {e_steps:.2e}")
        assert e <= 1.1 * e_steps, f"{k}: {e:.2e}, by steps {e_steps:.2e}"
        assert float((t.double() - ref[k]).abs().max()) <= 2 * float((steps[k].double() - ref[k]).abs().max()), k
