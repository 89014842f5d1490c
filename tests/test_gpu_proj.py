"""GPU parity of the linear maps around RSA (Table 2, rows Q/K/V and Linear) with the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check, download, upload
from paper_2105_13120_amd import inputs, rsa

pytestmark = pytest.mark.gpu


def draw(shape, seed, scale=1.0):
    x = np.random.Generator(np.random.PCG64(seed)).standard_normal(shape) * scale
    return inputs.round_to_bf16(x)


def check_f32(name, got, ref):
    """fp32 weight gradients: the bf16 products are exact in fp32, so the only error is the fp32
    accumulation over up to K/16 MFMA steps (K <= 16384 rows here): at most about 1000 roundings
    of 2^-24 relative to a partial sum of the size of the result, 6e-5 of its RMS if they all
    pointed the same way.  Bound: 2e-4 of the RMS, on the maximum error."""
    assert got.shape == ref.shape
    rms = float(np.sqrt(np.mean(np.square(ref))))
    err = float(np.abs(got - ref).max())
    assert err <= 2e-4 * rms, f"{name}: max abs err {err:.3e} vs rms {rms:.3e}"


# (B, Z, L, N, rank range, H, A): several 128-tiles, ragged 64-edges in M, N and K, one rank's share;
# heads of 64 and of 128 elements
CASES = [
    (1, 1, 64, 1, (0, 1), 64, 64),
    (2, 2, 128, 2, (0, 2), 192, 64),
    (1, 3, 320, 5, (0, 5), 320, 64),
    (2, 4, 512, 4, (1, 3), 256, 64),
    (1, 16, 2048, 8, (0, 8), 1024, 64),
    (1, 1, 64, 1, (0, 1), 64, 128),
    (2, 3, 320, 5, (1, 4), 192, 128),
    (2, 5, 512, 4, (0, 4), 320, 128),     # 15 column tiles per output: work-groups straddle Q | K | V
    (1, 8, 2048, 8, (0, 8), 1024, 128),
    (8, 16, 2048, 8, (0, 8), 1024, 64),   # the size bench.py times: 16384 rows, BERT Large's hidden size
]


@pytest.mark.parametrize("B,Z,L,N,ranks,H,A", CASES)
def test_projections_forward_and_backward(B, Z, L, N, ranks, H, A):
    rows = (ranks[1] - ranks[0]) * (L // N)
    X = draw((B, rows, H), 1)
    W = draw((H, 3 * Z * A), 2, H ** -0.5)
    Wo = draw((Z * A, H), 3, (Z * A) ** -0.5)
    O = draw((B, Z, rows, A), 4)
    dY = draw((B, rows, H), 5)
    dQ, dK, dV = (draw((B, Z, rows, A), s) for s in (6, 7, 8))
    t = {k: upload(v, "bf16") for k, v in dict(X=X, W=W, Wo=Wo, O=O, dY=dY, dQ=dQ, dK=dK, dV=dV).items()}
    Kfull = torch.empty((B, Z, L, A), dtype=torch.bfloat16, device="cuda")
    desc = rsa.make_desc(Kfull, N, rank_begin=ranks[0], rank_end=ranks[1])

    Q, K, V = rsa.qkv_proj(desc, t["X"], t["W"])
    Y = rsa.out_proj(desc, t["O"], t["Wo"])
    gO, gWo = rsa.out_proj_bwd(desc, t["dY"], t["O"], t["Wo"])
    gX, gW = rsa.qkv_proj_bwd(desc, t["dQ"], t["dK"], t["dV"], t["X"], t["W"])
    torch.cuda.synchronize()

    P = oracle.proj
    for name, got, ref in zip("QKV", (Q, K, V), P.qkv_proj(X, W, Z, A)):
        check(name, download(got), ref, "bf16")
    check("Y", download(Y), P.out_proj(O, Wo), "bf16")
    rO, rWo = P.out_proj_bwd(dY, O, Wo)
    check("dO", download(gO), rO, "bf16")
    check_f32("dWo", download(gWo), rWo)
    rX, rW = P.qkv_proj_bwd(dQ, dK, dV, X, W)
    check("dX", download(gX), rX, "bf16")
    check_f32("dWqkv", download(gW), rW)


def test_projection_outputs_feed_rsa_without_relayout():
    """X -> Q/K/V projection -> RSA -> Linear, against the oracle chain on the rounded intermediates."""
    B, Z, L, N, H, A = 1, 4, 512, 4, 256, 64
    X = draw((B, L, H), 11)
    W = draw((H, 3 * Z * A), 12, H ** -0.5)
    Wo = draw((Z * A, H), 13, (Z * A) ** -0.5)
    tX, tW, tWo = (upload(v, "bf16") for v in (X, W, Wo))
    Kfull = torch.empty((B, Z, L, A), dtype=torch.bfloat16, device="cuda")
    desc = rsa.make_desc(Kfull, N)
    Q, K, V = rsa.qkv_proj(desc, tX, tW)
    O, LSE = rsa.forward(desc, Q, K, V)
    Y = rsa.out_proj(desc, O, tWo)
    torch.cuda.synchronize()
    # the oracle continues from the GPU's rounded Q, K, V (each stage is checked on its own inputs)
    O_ref, _ = oracle.forward(download(Q), download(K), download(V))
    check("O", download(O), O_ref, "bf16")
    check("Y", download(Y), oracle.proj.out_proj(download(O), Wo), "bf16")


@pytest.mark.parametrize("Z,A", [(4, 64), (2, 128)])
def test_attention_block_backward_chain(Z, A):
    """dY -> Linear backward -> RSA backward -> Q/K/V projection backward: the whole block's
    gradients, each stage against the oracle on the rounded tensors that stage received."""
    B, L, N, H = 2, 512, 4, 256
    X = draw((B, L, H), 21)
    W = draw((H, 3 * Z * A), 22, H ** -0.5)
    Wo = draw((Z * A, H), 23, (Z * A) ** -0.5)
    dY = draw((B, L, H), 24)
    tX, tW, tWo, tdY = (upload(v, "bf16") for v in (X, W, Wo, dY))
    desc = rsa.make_desc(torch.empty((B, Z, L, A), dtype=torch.bfloat16), N)
    Q, K, V = rsa.qkv_proj(desc, tX, tW)
    O, LSE = rsa.forward(desc, Q, K, V)
    dO, dWo = rsa.out_proj_bwd(desc, tdY, O, tWo)
    dQ, dK, dV = rsa.backward(desc, dO, Q, K, V, O, LSE)
    dX, dW = rsa.qkv_proj_bwd(desc, dQ, dK, dV, tX, tW)
    torch.cuda.synchronize()
    P = oracle.proj
    rO, rWo = P.out_proj_bwd(dY, download(O), Wo)
    check("dO", download(dO), rO, "bf16")
    check_f32("dWo", download(dWo), rWo)
    g = oracle.backward(download(Q), download(K), download(V), download(dO))
    for name, got, ref in zip(("dQ", "dK", "dV"), (dQ, dK, dV), g):
        # O was rounded before D was formed from it, as in the kernels
        check(name, download(got), ref, "bf16")
    rX, rW = P.qkv_proj_bwd(download(dQ), download(dK), download(dV), X, W)
    check("dX", download(dX), rX, "bf16")
    check_f32("dWqkv", download(dW), rW)
    # and the block as a whole against fp64 end to end: errors of the stages compound,
    # so only the relative RMS error is held, to a few bf16 roundings
    fQ, fK, fV = P.qkv_proj(X, W, Z, A)
    fO, _ = oracle.forward(fQ, fK, fV)
    fdO, _ = P.out_proj_bwd(dY, fO, Wo)
    fg = oracle.backward(fQ, fK, fV, fdO)
    fdX, _ = P.qkv_proj_bwd(fg[0], fg[1], fg[2], X, W)
    err = download(dX) - fdX
    assert np.sqrt(np.mean(err ** 2)) <= 2e-2 * np.sqrt(np.mean(fdX ** 2))


def test_projection_error_codes():
    Kfull = torch.empty((1, 2, 128, 64), dtype=torch.bfloat16, device="cuda")
    desc = rsa.make_desc(Kfull, 2)
    X = torch.zeros((1, 128, 100), dtype=torch.bfloat16, device="cuda")   # H = 100: not a multiple of 64
    W = torch.zeros((100, 384), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(rsa.RSAError) as e:
        rsa.qkv_proj(desc, X, W)
    assert e.value.status == -3
    X = torch.zeros((1, 128, 128), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((128, 384), dtype=torch.bfloat16, device="cuda")
    g = torch.zeros((1, 2, 128, 64), dtype=torch.bfloat16, device="cuda")
    need = rsa.proj_workspace_bytes(desc, 128)
    if need > 0:
        with pytest.raises(rsa.RSAError) as e:
            rsa.qkv_proj_bwd(desc, g, g, g, X, W, ws=torch.empty(16, dtype=torch.uint8, device="cuda"))
        assert e.value.status == -4


# The size of the products chooses the work-groups' tiles: 64 x 64 with one and two groups of waves on k (an odd number
# of its slabs of 64 splits unevenly), 128 x 128, 256 x 256, each with ragged edges, and k splits of the weight gradients.
@pytest.mark.parametrize("B,Z,L,N,ranks,H,A", [
    (3, 5, 192, 1, (0, 1), 1216, 64),
    (2, 11, 256, 2, (0, 2), 1408, 128),
    (5, 9, 576, 3, (0, 3), 704, 64),
    (1, 3, 4224, 2, (1, 2), 1344, 128),
    (3, 4, 3008, 1, (0, 1), 320, 64),
    (6, 13, 1856, 1, (0, 1), 832, 64),
])
def test_projection_tile_sizes(B, Z, L, N, ranks, H, A):
    test_projections_forward_and_backward(B, Z, L, N, ranks, H, A)


@pytest.mark.parametrize("B,Z,L,H,A", [
    (8, 16, 2048, 1024, 64),    # dWo 1024 x 1024 over 16384 rows
    (16, 12, 512, 768, 64),
    (4, 8, 960, 512, 128),
    (1, 31, 4160, 448, 64),     # a number of slabs that no chain divides
])
def test_weight_gradients_are_summed_in_short_chains(B, Z, L, H, A):
    """fp32 weight gradients over K rows: a chain of additions is as long as splitting K until every CU has a 256 x 256
    tile leaves it (at most 64 splits of at least 256 rows), however the kernel cuts the product.  The matrix core adds
    16 products at a time, so a chain of n rows rounds n / 16 times at partial sums that grow with the root, and the
    K / n chains once each: RMS error u sqrt(n / 32 + K / 2n) of the result's RMS, u = 0.55 * 2^-24 the RMS of one
    rounding.  1.25 times that is allowed (measured 0.7 to 1.05 of the formula; chains up to four times as long: 1.4 to 2)."""
    K, D = B * L, Z * A
    g = torch.Generator(device="cuda").manual_seed(5)
    mk = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    X, dY, W, Wo, O, dQ, dK, dV = (mk(B, L, H), mk(B, L, H), mk(H, 3 * D), mk(D, H)) + tuple(mk(B, Z, L, A) for _ in range(4))
    desc = rsa.make_desc(O, 1)
    rows = lambda t: t.permute(0, 2, 1, 3).reshape(K, D).double()
    _, dWo = rsa.out_proj_bwd(desc, dY, O, Wo)
    _, dW = rsa.qkv_proj_bwd(desc, dQ, dK, dV, X, W)
    ref = rows(O).T.contiguous() @ dY.reshape(K, H).double()
    ref3 = X.reshape(K, H).double().T.contiguous() @ torch.cat([rows(t) for t in (dQ, dK, dV)], 1)
    for name, got, r in (("dWo", dWo, ref), ("dWqkv", dW, ref3)):
        tiles = -(-r.shape[0] // 256) * -(-r.shape[1] // 256)
        splits = max(1, min(64, 256 // tiles, K // 64 // 4))
        n = 64 * -(-(K // 64) // splits)
        bound = 1.25 * 0.55 * 2.0 ** -24 * np.sqrt(n / 32 + K / n / 2)
        err = float((got.double() - r).norm() / r.norm())
        assert err <= bound, f"{name}: {err:.2e} > {bound:.2e}"


def test_rows_longer_than_32_bits_of_offset():
    """H = 35 * 2^20: the rows of a tile span more than 2^32 bytes, those of half a tile more than 2^31, in operands read
    along their rows (X, dY, Wo for dO) and across them (Wo for Y, dY for dWo)."""
    H, A, edge = 35 << 20, 64, 1024
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(3)
    mk = lambda *s: torch.randn(s, generator=g, device=dev).bfloat16()
    ends = lambda t, d: torch.cat((t.narrow(d, 0, edge), t.narrow(d, H - edge, edge)), d).float()

    def edges(*s, dim):       # zero but for the first and last rows or columns: contractions over H are these alone
        t = torch.zeros(s, dtype=torch.bfloat16, device=dev)
        for at in (0, H - edge):
            t.narrow(dim, at, edge).copy_(mk(*(edge if k == dim else n for k, n in enumerate(s))))
        return t

    def close(got, ref, tol=3e-3):                     # one rounding to bf16
        assert float((got.float() - ref).norm() / ref.norm()) <= tol

    O = mk(1, 1, 64, A)
    desc = rsa.make_desc(O, 1)
    X, W = edges(1, 64, H, dim=2), edges(H, 3 * A, dim=0)
    close(torch.cat(rsa.qkv_proj(desc, X, W), -1)[0, 0], ends(X[0], 1) @ ends(W, 0))
    dY, Wo = X, torch.stack([mk(H) for _ in range(A)])
    del X, W
    dO, dWo = rsa.out_proj_bwd(desc, dY, O, Wo)
    close(dO[0, 0], ends(dY[0], 1) @ ends(Wo, 1).T)
    close(ends(dWo, 1), O[0, 0].float().T @ ends(dY[0], 1), 1e-6)   # fp32, 64 products each
    del dO, dWo, dY
    Y = rsa.out_proj(desc, O, Wo)
    for at in (0, H // 2, H - (1 << 20)):
        close(Y[0].narrow(1, at, 1 << 20), O[0, 0].float() @ Wo.narrow(1, at, 1 << 20).float())
