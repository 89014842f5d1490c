"""GPU parity of the fused (online-softmax) RSA kernels against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from helpers import (BF16_REL_RMS, LSE_ATOL, check, compare_heads, download, gpu_forward_backward,
                     heads_view, rel_rms_err, upload)
from paper_2105_13120_amd import inputs, rsa

pytestmark = pytest.mark.gpu


def cfg_of(B, Z, L, N, causal=False, rb=0, re=-1, seed=7, scale=1.0, zigzag=False, A=64, att_scale=0.0):
    return inputs.RSAConfig("t", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal,
                            rank_begin=rb, rank_end=re, seed=seed, qkv_scale=scale, zigzag=zigzag,
                            att_scale=att_scale)


# sizes that span several 64-key tiles, several work-groups and ragged tails
# (Lq not a multiple of the 128/256-row work-group tile, L not a multiple of 256)
SHAPES = [
    (1, 1, 64, 1), (1, 2, 128, 2), (2, 3, 320, 5), (1, 2, 448, 7), (1, 2, 1024, 4),
    (1, 1, 1536, 3),
]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Z,L,N", SHAPES)
def test_fused_forward_backward_whole_ring(B, Z, L, N, causal):
    cfg = cfg_of(B, Z, L, N, causal)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    compare_heads(cfg, x, out, list(range(B * Z)))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Z,L,N,rb,re,zigzag", [
    (1, 1, 64, 1, 0, -1, False), (2, 3, 320, 5, 0, -1, False), (1, 2, 1024, 4, 0, -1, False),
    (1, 2, 640, 5, 1, 4, False),     # three ranks of five: partial dK, dV
    (1, 2, 1024, 4, 0, -1, True),    # zig-zag ownership, whole ring
    (1, 2, 1536, 3, 1, 2, True),     # zig-zag, one rank's share
    (1, 2, 4096, 4, 3, 4, False),    # split key walk
    (1, 1, 4096, 2, 0, 1, True),     # split key walk under zig-zag ownership
])
def test_heads_of_128(B, Z, L, N, rb, re, zigzag, causal):
    """A = 128: the fused kernels take a head as two halves of 64."""
    cfg = cfg_of(B, Z, L, N, causal, rb=rb, re=re, seed=53, zigzag=zigzag, A=128)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    compare_heads(cfg, x, out, list(range(B * Z)))


@pytest.mark.parametrize("A,att_scale", [(64, 0.2), (64, 0.07), (128, 0.11)])
@pytest.mark.parametrize("causal,rb,re", [(False, 0, -1), (True, 0, -1), (True, 3, 4)])
def test_explicit_softmax_scale(A, att_scale, causal, rb, re):
    """rsa_desc.scale other than 1/sqrt(A), and not a power of two: it enters the scores, the LSE
    and the factors of dQ and dK."""
    cfg = cfg_of(1, 2, 1024, 4, causal, rb=rb, re=re, seed=71, A=A, att_scale=att_scale)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    compare_heads(cfg, x, out, [0, 1])
    # the default would have given something else
    ref = gpu_forward_backward(cfg_of(1, 2, 1024, 4, causal, rb=rb, re=re, seed=71, A=A), x)
    assert not torch.equal(out["O"], ref["O"])


@pytest.mark.parametrize("A", [64, 128])
@pytest.mark.parametrize("causal,rb,re,zigzag", [(False, 0, -1, False), (True, 0, -1, True), (True, 3, 4, False)])
def test_strided_layouts(A, causal, rb, re, zigzag):
    """Q, K, V as slices of one packed projection output (B, rows, 3, Z, A), O and dO with the heads
    interleaved (B, rows, Z, A) -- the layouts the linear maps either side of RSA produce and consume
    without a transpose -- and dQ, dK, dV written back into a packed buffer.  The strides travel in
    the descriptor; the results are those of the dense layout bit for bit."""
    B, Z, L, N = 2, 3, 2048, 4
    cfg = cfg_of(B, Z, L, N, causal, rb=rb, re=re, seed=83, zigzag=zigzag, A=A)
    x = inputs.make_inputs(cfg)
    dense = {k: upload(x[k], "bf16") for k in ("Q", "K", "V", "dO")}
    Lq = cfg.Lq
    # packed (B, L, 3, Z, A): Q lives in slot 0 of the first Lq rows (a rank share has fewer query rows)
    packed = torch.zeros((B, L, 3, Z, A), dtype=torch.bfloat16, device="cuda")
    view = lambda t, i, rows: t[:, :rows, i].permute(0, 2, 1, 3)          # (B, Z, rows, A), not contiguous
    Q, K, V = view(packed, 0, Lq), view(packed, 1, L), view(packed, 2, L)
    Q.copy_(dense["Q"]); K.copy_(dense["K"]); V.copy_(dense["V"])
    inter = lambda: torch.full((B, Lq, Z, A), float("nan"), dtype=torch.bfloat16, device="cuda").permute(0, 2, 1, 3)
    O, dO = inter(), inter()
    dO.copy_(dense["dO"])
    grads = torch.full_like(packed, float("nan"))
    dQ, dK, dV = view(grads, 0, Lq), view(grads, 1, L), view(grads, 2, L)
    assert not Q.is_contiguous() and not O.is_contiguous()
    kw = dict(causal=causal, rank_begin=cfg.ranks[0], rank_end=cfg.ranks[1], zigzag=zigzag)
    desc = rsa.make_desc(K, N, Q=Q, O=O, **kw)
    LSE = torch.empty((B, Z, Lq), dtype=torch.float32, device="cuda")
    rsa.forward(desc, Q, K, V, O=O, LSE=LSE)
    rsa.backward(desc, dO, Q, K, V, O, LSE, dQ=dQ, dK=dK, dV=dV)
    # the dense layout through the same kernels
    ddesc = rsa.make_desc(dense["K"], N, **kw)
    O2, LSE2 = rsa.forward(ddesc, dense["Q"], dense["K"], dense["V"])
    g2 = rsa.backward(ddesc, dense["dO"], dense["Q"], dense["K"], dense["V"], O2, LSE2)
    torch.cuda.synchronize()
    for name, a, b in (("O", O, O2), ("LSE", LSE, LSE2), ("dQ", dQ, g2[0]), ("dK", dK, g2[1]), ("dV", dV, g2[2])):
        assert torch.equal(a.contiguous(), b), name
    # nothing outside the views was written: the unused slots of the packed gradient stay NaN
    if Lq < L:
        assert torch.isnan(grads[:, Lq:, 0]).all()
    out = dict(O=O.contiguous(), LSE=LSE, dQ=dQ.contiguous(), dK=dK.contiguous(), dV=dV.contiguous())
    compare_heads(cfg, x, out, list(range(B * Z)))


def test_kernel_error_matches_the_model_of_its_roundings():
    """The ideal bf16 pipeline (tests/bf16_model.py) makes exactly the roundings the fused kernels
    make, so on the same inputs the two errors agree as distributions: RMS within 10 % and the
    99.9th percentile within 20 %, from both sides (compare_heads holds only the upper side)."""
    for causal in (False, True):
        cfg = cfg_of(1, 4, 1024, 4, causal, seed=0)
        x = inputs.make_inputs(cfg)
        errs = compare_heads(cfg, x, gpu_forward_backward(cfg, x), [0, 1, 2, 3])
        for name in ("O", "dQ", "dK", "dV"):
            e = errs[name]
            assert 0.9 <= e.vs_ideal_rms <= 1.1, (name, causal, e.describe())
            assert 0.8 <= e.vs_ideal_p999 <= 1.2, (name, causal, e.describe())


def test_heads_of_128_backward_parts_equal_the_whole():
    cfg = cfg_of(1, 2, 512, 4, causal=True, seed=59, A=128)
    x = inputs.make_inputs(cfg)
    Q, K, V, dO = (upload(x[k], "bf16") for k in ("Q", "K", "V", "dO"))
    desc = rsa.make_desc(K, cfg.N, causal=True)
    O, LSE = rsa.forward(desc, Q, K, V)
    ws = torch.empty(rsa.workspace_bytes(desc, True), dtype=torch.uint8, device="cuda")
    dQ, dK, dV = torch.empty_like(Q), torch.empty_like(K), torch.empty_like(V)
    rsa.bwd_preprocess(desc, dO, O, LSE, ws)
    rsa.bwd_dkdv(desc, dO, Q, K, V, ws, dK, dV)
    rsa.bwd_dq(desc, dO, Q, K, V, ws, dQ)
    torch.cuda.synchronize()
    compare_heads(cfg, x, dict(O=O, LSE=LSE, dQ=dQ, dK=dK, dV=dV), [0, 1])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("rb,re", [(0, 1), (2, 3), (4, 5), (1, 4)])
def test_fused_rank_subrange_gives_partial_sums(causal, rb, re):
    cfg = cfg_of(1, 2, 640, 5, causal, rb=rb, re=re, seed=9)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    compare_heads(cfg, x, out, [0, 1])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Z,L,N,rb,re,zigzag", [
    (1, 2, 4096, 4, 3, 4, False),    # last rank of four: every split of the key walk has work
    (1, 2, 8192, 8, 0, 2, False),    # first ranks: under the mask only their own chunks are visible (no split)
    (1, 1, 8192, 16, 4, 10, False),  # six ranks, ring walks that wrap around
    (1, 2, 4096, 2, 0, 1, True),     # zig-zag share: its first half sees few keys, its second all
    (1, 1, 6144, 3, 1, 2, True),     # odd ring size, 3 splits
    (1, 1, 4608, 9, 8, 9, False),    # 36 stages in 2 splits: the boundary falls inside a chunk
    (1, 1, 4224, 11, 10, 11, False), # chunks of 6 tiles
    (1, 1, 6336, 33, 32, 33, False), # chunks of 3 tiles: one tile per stage, 49 stages in 3 splits
])
def test_split_key_walk(B, Z, L, N, rb, re, zigzag, causal):
    """Few query rows against many keys: the forward and dQ kernels divide the walk over the keys
    among several work-groups per row tile and merge their partial results."""
    cfg = cfg_of(B, Z, L, N, causal, rb=rb, re=re, seed=43, zigzag=zigzag)
    desc = rsa.make_desc(torch.empty(B, Z, L, 64, dtype=torch.bfloat16), N, causal=causal,
                         rank_begin=rb, rank_end=re, zigzag=zigzag)
    # the split is on for these shapes, except where the mask hides most of the keys
    assert (rsa.workspace_bytes(desc, False) > 0) == (not (causal and rb == 0 and not zigzag))
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    compare_heads(cfg, x, out, list(range(B * Z)))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("rb,zigzag", [(15, False), (0, True), (3, True)])
def test_split_key_walk_with_256_row_tiles(rb, zigzag, causal):
    """Enough heads and keys that the split forward takes its 256-row work-groups
    (16 heads x 4 row tiles x 8 splits = 512 work-groups)."""
    cfg = cfg_of(2, 8, 16384, 16, causal, rb=rb, re=rb + 1, seed=47, zigzag=zigzag)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    compare_heads(cfg, x, out, [0, 6, 15])


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Z,L,N,rb,re", [
    (1, 2, 512, 4, 0, -1),      # whole ring, half-chunks of 64 rows
    (1, 2, 1024, 4, 0, -1),     # half-chunks of 128 rows: two tiles per stage
    (2, 2, 768, 3, 0, -1),      # odd ring size
    (1, 2, 1536, 3, 1, 2),      # one rank's share (work-group straddles its two half-chunks)
    (1, 1, 2048, 4, 3, 4),      # last rank: half-chunks 3 and 4 are neighbours
    (1, 2, 1280, 5, 1, 4),      # three ranks of five
    (1, 1, 4096, 2, 0, 1),      # half-chunks of 1024 rows: whole work-groups inside one half
])
def test_zigzag_ownership(B, Z, L, N, rb, re, causal):
    """Rank n holds tokens of half-chunks n and 2N-1-n; the oracle is called once per run of
    consecutive tokens and the runs' partial dK, dV are added."""
    cfg = cfg_of(B, Z, L, N, causal, rb=rb, re=re, seed=13, zigzag=True)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    compare_heads(cfg, x, out, list(range(B * Z)))


@pytest.mark.parametrize("B,Z,L,N,rb,re,causal", [
    (1, 73, 1600, 5, 0, 5, False),     # the last work-group of a head holds 64 rows,
    (6, 17, 1152, 3, 0, 3, False),     # 128,
    (25, 8, 1472, 1, 0, 1, False),     # 192
    (8, 38, 896, 2, 1, 2, False),      # one rank's 448
    (5, 12, 4416, 3, 0, 3, True),      # causal
])
def test_forward_ragged_256_row_tiles(B, Z, L, N, rb, re, causal):
    """Work-groups of 256 rows whose last one of a head is in part not there."""
    cfg = cfg_of(B, Z, L, N, causal, rb=rb, re=re, seed=23)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x, backward=False)
    compare_heads(cfg, x, out, [0, B * Z - 1], backward=False)


@pytest.mark.parametrize("A", [64, 128])
@pytest.mark.parametrize("B,Z,L,N,rb,re", [
    (1, 2, 1920, 5, 1, 4),      # h of three tiles: work-groups' rows from the ends of two ranks' half-chunks, a gap of tokens
    (5, 13, 1920, 5, 0, 5),     # one group of waves
    (2, 9, 4480, 7, 2, 6),      # longer walks, groups of waves
])
def test_zigzag_rows_by_token(A, B, Z, L, N, rb, re):
    """Half-chunks of an odd number of 64-row tiles: work-groups take rows in the order of their tokens, across ranks."""
    cfg = cfg_of(B, Z, L, N, True, rb=rb, re=re, seed=19, zigzag=True, A=A)
    x = inputs.make_inputs(cfg)
    compare_heads(cfg, x, gpu_forward_backward(cfg, x), [0, B * Z - 1])


def test_zigzag_whole_ring_is_a_row_permutation_of_the_contiguous_ring():
    """Ownership only decides which rank holds a row: over the whole ring the outputs are
    those of the contiguous layout, rows permuted (different summation order: tolerance)."""
    cfg = cfg_of(1, 2, 1024, 4, True, seed=17)
    zz = cfg_of(1, 2, 1024, 4, True, seed=17, zigzag=True)
    x = inputs.make_inputs(cfg)
    perm = np.concatenate([np.arange(t0, t0 + n) for _, t0, n in zz.segments()])
    xz = dict(x, Q=np.ascontiguousarray(x["Q"][:, :, perm]), dO=np.ascontiguousarray(x["dO"][:, :, perm]))
    a = {k: download(v) for k, v in gpu_forward_backward(cfg, x).items()}
    b = {k: download(v) for k, v in gpu_forward_backward(zz, xz).items()}
    check("O", b["O"], a["O"][:, :, perm], "bf16", both_rounded=True)
    check("dQ", b["dQ"], a["dQ"][:, :, perm], "bf16", both_rounded=True)
    check("dK", b["dK"], a["dK"], "bf16", both_rounded=True)
    check("dV", b["dV"], a["dV"], "bf16", both_rounded=True)
    assert np.abs(b["LSE"] - a["LSE"][:, :, perm]).max() <= LSE_ATOL


def test_result_is_independent_of_the_ring_size():
    """Eq. 3 is a block decomposition: any N dividing L gives the same attention."""
    base = cfg_of(1, 2, 1024, 1, seed=5)
    x = inputs.make_inputs(base)
    ref = None
    for N in (1, 2, 4, 8, 16):
        cfg = cfg_of(1, 2, 1024, N, seed=5)
        out = {k: download(v) for k, v in gpu_forward_backward(cfg, x).items()}
        if ref is None:
            ref = out
            compare_heads(cfg, x, gpu_forward_backward(cfg, x), [0, 1])
        else:
            for k in ("O", "dQ", "dK", "dV"):
                check(k, out[k], ref[k], "bf16", both_rounded=True)
            assert np.abs(out["LSE"] - ref["LSE"]).max() <= LSE_ATOL


def test_invariants_on_gpu_output():
    cfg = cfg_of(1, 2, 512, 4, seed=13)
    x = inputs.make_inputs(cfg)
    x["V"] = np.ones_like(x["V"])
    out = gpu_forward_backward(cfg, x)
    assert np.abs(download(out["O"]) - 1.0).max() <= 2 ** -8      # rows of P sum to 1
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    dK, dV = download(out["dK"]), download(out["dV"])
    scale = np.sqrt(np.mean(dK ** 2)) * np.sqrt(cfg.L)
    assert np.abs(dK.sum(2)).max() <= 0.05 * scale                # sum_j dK_j = 0
    ref = x["dO"].astype(np.float64).sum(2)
    assert np.abs(dV.sum(2) - ref).max() <= 0.02 * np.abs(ref).max() + 0.5


def test_growing_scores_exercise_the_lazy_rescale():
    """Key magnitude grows along the sequence, so later tiles raise the running row
    max by more than the 2^8 slack and the accumulators are rescaled several times."""
    cfg = cfg_of(1, 2, 768, 3, seed=17)
    x = inputs.make_inputs(cfg)
    ramp = np.linspace(0.2, 2.0, cfg.L, dtype=np.float32)[None, None, :, None]
    x["Q"] = inputs.round_to_bf16(x["Q"] * 2.0)
    x["K"] = inputs.round_to_bf16(x["K"] * ramp)      # score std from 0.4 to 4 along the keys
    S = oracle.forward(x["Q"].astype(np.float64), x["K"].astype(np.float64),
                       x["V"].astype(np.float64), want_scores=True)[2]
    tile_max = S.reshape(1, 2, 768, 12, 64).max(-1)
    running = np.maximum.accumulate(tile_max, axis=-1)
    jumps = (np.diff(running, axis=-1) > 8 * np.log(2)).sum()
    assert jumps > 20            # rows whose max jumps by more than 2^8 between tiles exist
    # Forward only: the rescale lives in the forward kernel, and with scores this
    # spread the backward is ill-conditioned for bf16 operands (an exact pipeline
    # that only rounds P, dS and O to bf16 is 5e-2 of the RMS off on these inputs).
    for causal in (False, True):
        c2 = cfg_of(1, 2, 768, 3, causal=causal, seed=17)
        out = gpu_forward_backward(c2, x, backward=False)
        compare_heads(c2, x, out, [0, 1], backward=False)


def test_staged_and_fused_agree():
    cfg = cfg_of(2, 2, 512, 4, seed=19)
    x = inputs.make_inputs(cfg)
    a = gpu_forward_backward(cfg, x, mode=rsa.MODE_FUSED)
    b = gpu_forward_backward(cfg, x, mode=rsa.MODE_STAGED)
    for k in ("O", "dQ", "dK", "dV"):
        check(k, download(a[k]), download(b[k]), "bf16", both_rounded=True)


def test_fused_path_is_deterministic():
    """No atomics anywhere: two runs on the same inputs give the same bits."""
    cfg = cfg_of(2, 2, 768, 3, causal=True, seed=23)
    x = inputs.make_inputs(cfg)
    a = gpu_forward_backward(cfg, x)
    b = gpu_forward_backward(cfg, x)
    for k in ("O", "LSE", "dQ", "dK", "dV"):
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("causal", [False, True])
def test_chunk_of_64_rows_and_single_rank_of_many(causal):
    """Smallest chunk (c = 64, N = 16) for the whole ring, and one middle rank of it."""
    for rb, re in ((0, -1), (7, 8)):
        cfg = cfg_of(1, 2, 1024, 16, causal=causal, rb=rb, re=re, seed=29)
        x = inputs.make_inputs(cfg)
        out = gpu_forward_backward(cfg, x)
        compare_heads(cfg, x, out, [0, 1])


def test_outputs_do_not_depend_on_buffer_contents():
    """dQ, dK, dV, O are overwritten, not accumulated into (buffers pre-filled with NaN)."""
    cfg = cfg_of(1, 2, 384, 3, seed=31)
    x = inputs.make_inputs(cfg)
    Q, K, V, dO = (upload(x[k], "bf16") for k in ("Q", "K", "V", "dO"))
    desc = rsa.make_desc(K, cfg.N)
    nan = lambda t: torch.full_like(t, float("nan"))
    O, LSE = rsa.forward(desc, Q, K, V, O=nan(Q), LSE=torch.full(Q.shape[:3], float("nan"), device="cuda"))
    ws = torch.full((rsa.workspace_bytes(desc, True),), 0xFF, dtype=torch.uint8, device="cuda")
    dQ, dK, dV = rsa.backward(desc, dO, Q, K, V, O, LSE, dQ=nan(Q), dK=nan(K), dV=nan(V), ws=ws)
    torch.cuda.synchronize()
    compare_heads(cfg, x, dict(O=O, LSE=LSE, dQ=dQ, dK=dK, dV=dV), [0, 1])


def test_backward_parts_equal_the_whole():
    """rsa_bwd_preprocess + rsa_bwd_dkdv + rsa_bwd_dq against rsa_backward, which folds the
    preprocess into the dQ kernel: the same gradients up to the fp32 summation order of D
    (a last-bit difference in D moves an occasional bf16 output by one ulp)."""
    cfg = cfg_of(1, 3, 512, 4, causal=True, seed=37)
    x = inputs.make_inputs(cfg)
    Q, K, V, dO = (upload(x[k], "bf16") for k in ("Q", "K", "V", "dO"))
    desc = rsa.make_desc(K, cfg.N, causal=True)
    O, LSE = rsa.forward(desc, Q, K, V)
    dQ, dK, dV = rsa.backward(desc, dO, Q, K, V, O, LSE)
    ws = torch.empty(rsa.workspace_bytes(desc, True), dtype=torch.uint8, device="cuda")
    dQ2, dK2, dV2 = torch.empty_like(Q), torch.empty_like(K), torch.empty_like(V)
    rsa.bwd_preprocess(desc, dO, O, LSE, ws)
    rsa.bwd_dkdv(desc, dO, Q, K, V, ws, dK2, dV2)
    rsa.bwd_dq(desc, dO, Q, K, V, ws, dQ2)
    torch.cuda.synchronize()
    for name, a, b in (("dQ", dQ, dQ2), ("dK", dK, dK2), ("dV", dV, dV2)):
        a, b = download(a), download(b)
        rms = np.sqrt(np.mean(a * a))
        assert np.abs(a - b).max() <= 2.0 ** -7 * np.abs(a).max() + 1e-30, name   # within one bf16 ulp
        assert np.sqrt(np.mean((a - b) ** 2)) <= 1e-3 * rms, name
    compare_heads(cfg, x, dict(O=O, LSE=LSE, dQ=dQ2, dK=dK2, dV=dV2), [0, 1, 2])


def test_error_codes_on_the_device_path():
    cfg = cfg_of(1, 1, 128, 2, seed=41)
    x = inputs.make_inputs(cfg)
    Q, K, V = (upload(x[k], "bf16") for k in ("Q", "K", "V"))
    desc = rsa.make_desc(K, 3)                      # 128 % 3 != 0
    with pytest.raises(rsa.RSAError) as e:
        rsa.forward(desc, Q, K, V)
    assert e.value.status == -2
    desc = rsa.make_desc(K, 2)
    O, LSE = rsa.forward(desc, Q, K, V)
    with pytest.raises(rsa.RSAError) as e:          # backward workspace too small
        rsa.backward(desc, Q, Q, K, V, O, LSE, ws=torch.empty(64, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -4
