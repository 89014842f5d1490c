"""The fused backward's dQ and dK, dV work-groups in one grid: every work-group shape the launch rule picks from, at sizes
with ragged tiles and counts that do not divide by the eights the work-groups are dealt out in."""
import numpy as np
import pytest
import torch

from helpers import compare_heads, download, gpu_forward_backward, upload
from paper_2105_13120_amd import inputs, rsa

pytestmark = pytest.mark.gpu

# (A, B, Z, L, N, first rank, last rank + 1, causal, zig-zag)
CASES = [
    (64, 1, 1, 64, 1, 0, 1, False, False), (64, 1, 3, 1088, 17, 0, 17, True, False), (64, 1, 2, 2048, 4, 0, 4, False, False),
    (64, 2, 5, 448, 7, 0, 7, False, False), (64, 1, 9, 1024, 4, 0, 4, True, True), (64, 5, 8, 320, 5, 0, 5, True, False),
    (64, 3, 11, 512, 4, 0, 4, False, False), (64, 1, 19, 1728, 3, 0, 3, True, False), (64, 3, 25, 704, 11, 0, 11, True, False),
    (64, 1, 7, 1024, 4, 1, 3, True, False), (64, 1, 5, 768, 6, 2, 3, False, False),       # a share of the rows
    (128, 1, 3, 704, 11, 0, 11, True, False), (128, 2, 9, 576, 9, 0, 9, False, False), (128, 1, 17, 1024, 4, 0, 4, True, True),
]


@pytest.mark.parametrize("A,B,Z,L,N,rb,re,causal,zigzag", CASES)
def test_against_the_oracle_and_the_kernels_one_by_one(A, B, Z, L, N, rb, re, causal, zigzag):
    cfg = inputs.RSAConfig("g", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=rb, rank_end=re, seed=41,
                           zigzag=zigzag)
    x = inputs.make_inputs(cfg)
    out = gpu_forward_backward(cfg, x)
    compare_heads(cfg, x, out, sorted({0, B * Z // 2, B * Z - 1}))
    Q, K, V, dO = (upload(x[k], "bf16") for k in ("Q", "K", "V", "dO"))
    desc = rsa.make_desc(K, N, causal=causal, rank_begin=rb, rank_end=re, zigzag=zigzag)
    ws = torch.empty(rsa.workspace_bytes(desc, True), dtype=torch.uint8, device="cuda")
    one = dict(dQ=torch.empty_like(Q), dK=torch.empty_like(K), dV=torch.empty_like(V))
    rsa.bwd_preprocess(desc, dO, out["O"], out["LSE"], ws)
    rsa.bwd_dkdv(desc, dO, Q, K, V, ws, one["dK"], one["dV"])
    rsa.bwd_dq(desc, dO, Q, K, V, ws, one["dQ"])
    torch.cuda.synchronize()
    for name, t in one.items():
        a, b = download(out[name]), download(t)
        # the same products in another order of the fp32 sums: an element's bf16 may round the other way
        assert (np.abs(a - b) <= 2.0 ** -7 * np.abs(b) + 1e-4 * np.sqrt(np.mean(b * b))).all(), name
        assert np.sqrt(np.mean((a - b) ** 2)) <= 1e-3 * np.sqrt(np.mean(b * b)), name


@pytest.mark.parametrize("A,B,Z,L,N,causal", [(64, 1, 3, 1088, 17, True), (64, 3, 11, 512, 4, False), (128, 2, 9, 576, 9, False),
                                              (64, 16, 8, 1024, 4, False)])
@pytest.mark.parametrize("dk,dv", [("K", "V"), ("V", "K"), ("K", None), (None, "K")])
def test_gradients_over_keys_and_values(A, B, Z, L, N, causal, dk, dv):
    """dK and dV may lie exactly over K and V: the two kinds then take turns, the gradients are those of buffers of their
    own (to the order of the fp32 sums, see above)."""
    cfg = inputs.RSAConfig("g", B=B, Z=Z, L=L, A=A, N=N, dtype="bf16", causal=causal, rank_begin=0, rank_end=N, seed=47)
    x = inputs.make_inputs(cfg)
    t = {k: upload(x[k], "bf16") for k in ("Q", "K", "V", "dO")}
    desc = rsa.make_desc(t["K"], N, causal=causal)
    O, LSE = rsa.forward(desc, t["Q"], t["K"], t["V"])
    ref = [download(g) for g in rsa.backward(desc, t["dO"], t["Q"], t["K"], t["V"], O, LSE)]
    got = rsa.backward(desc, t["dO"], t["Q"], t["K"], t["V"], O, LSE, dK=t.get(dk), dV=t.get(dv))
    for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
        a = download(a)
        assert (np.abs(a - b) <= 2.0 ** -7 * np.abs(b) + 1e-4 * np.sqrt(np.mean(b * b))).all(), name
        assert np.sqrt(np.mean((a - b) ** 2)) <= 1e-3 * np.sqrt(np.mean(b * b)), name
