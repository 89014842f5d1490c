"""The gradients of the maps around RSA formed in one grid: sizes at which each combination of tiles is taken, with
ragged tiles of every size, k splits of the weight gradient, heads of 128, and the calls that keep two launches."""
import pytest
import torch

from paper_2105_13120_amd import rsa

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -8  # one rounding to bf16


def close(x, ref, bound, k, f32=False):
    """An element is a sum of k exact products: its error is at most k roundings of the sum of their magnitudes in fp32
    (2^-24 each, far less in effect), and one rounding to bf16 where it is stored as such.  Over all elements, with one
    rounding of at most 2^-24 after every 8 of k, of partial sums that grow with the root of their length, the RMS error is
    2^-24 sqrt(k / 16 + 1) of the RMS at most; as much again is allowed for the sums of splits and folds.  (Partial sums kept in
    bf16 or one of 16384 rows left out: 1000 times that.)  A rounding to bf16: 2^-9 at most."""
    err = (x.double() - ref).abs()
    assert float(err.norm()) <= (2.0 ** -23 * (k / 16 + 1) ** 0.5 + (0 if f32 else EPS / 2)) * float(ref.norm())
    tol = bound * (k * 2.0 ** -24) + (0 if f32 else EPS * ref.abs()) + 1e-30
    assert bool((err <= tol).all()), float((err / tol).max())


def rand(*shape):
    return torch.randn(*shape, device="cuda").bfloat16()


def heads_to_rows(x):  # (B, Z, L, A) -> (B L, Z A), in 64 bits
    B, Z, L, A = x.shape
    return x.double().permute(0, 2, 1, 3).reshape(B * L, Z * A)


def check(rows, Z, A, H, in_place=False):
    torch.manual_seed(rows + H)
    d = rsa.make_desc(torch.empty(1, Z, rows, A, device="cuda", dtype=torch.bfloat16), 1)
    g = [rand(1, Z, rows, A) for _ in range(3)]
    X, W, Wo, dY = rand(1, rows, H), rand(H, 3 * Z * A), rand(Z * A, H), rand(1, rows, H)
    cat = torch.cat([heads_to_rows(t) for t in g], 1)
    Xd, Wd, dYd, Wod = X[0].double(), W.double(), dY[0].double(), Wo.double()
    dW = None
    if in_place:  # fp32 gradients whose first half is the weights themselves
        dW = torch.empty(H, 3 * Z * A, device="cuda")
        flat = dW.view(torch.bfloat16).flatten()[:W.numel()]
        flat.copy_(W.flatten())
        W = flat.view_as(W)
    dX, dW = rsa.qkv_proj_bwd(d, *g, X, W, dW=dW)
    close(dX[0], cat @ Wd.T, cat.abs() @ Wd.abs().T, 3 * Z * A)
    close(dW, Xd.T @ cat, Xd.abs().T @ cat.abs(), rows, f32=True)
    dO, dWo = rsa.out_proj_bwd(d, dY, g[0], Wo)
    O = heads_to_rows(g[0])
    close(heads_to_rows(dO), dYd @ Wod.T, dYd.abs() @ Wod.abs().T, H)
    close(dWo, O.T @ dYd, O.abs().T @ dYd.abs(), rows, f32=True)


@pytest.mark.parametrize("rows,Z,A,H", [
    (64, 1, 64, 64),        # one tile
    (192, 5, 64, 448),      # tiles of 64, in groups; ragged tiles of 128 and 256
    (1024, 3, 128, 960),
    (1536, 19, 64, 1216),   # two launches; tiles of 128
    (2048, 6, 128, 704),    # tiles of 128; beside tiles of 64 in two groups
    (3072, 19, 64, 1216),
    (8256, 16, 64, 1088),   # the weight gradient in k splits
    (16384, 16, 64, 1024),  # tiles of 256 beside tiles of 128 in two groups
    (64, 16, 64, 1024),     # tiles of 64 in two groups beside tiles of 128
    (1344, 2, 64, 3072),    # tiles of 256 beside tiles of 128 in two groups, no split
    (16384, 7, 64, 448),    # tiles of 256, in k splits
    (8256, 2, 128, 1920),
])
def test_maps(rows, Z, A, H):
    check(rows, Z, A, H)


def test_weight_gradient_over_the_weights():
    check(320, 4, 64, 256, in_place=True)


@pytest.mark.parametrize("rows,Z,A,Kp,over", [
    (64, 1, 64, 64, False),
    (896, 6, 64, 128, False),     # tiles of 64
    (6272, 5, 128, 128, False),   # tiles of 128 beside tiles of 64
    (13312, 18, 64, 128, False),  # tiles of 128
    (4160, 14, 64, 512, False),
    (19136, 7, 64, 512, False),
    (896, 6, 64, 128, True),      # dX over X: two launches
    (19136, 3, 64, 320, False),   # tiles of 256
    (19136, 2, 128, 256, False),
    (7296, 27, 64, 256, False),   # tiles of 128, close to the line between one grid and two launches
])
def test_projection_along_the_sequence(rows, Z, A, Kp, over):
    torch.manual_seed(rows + Kp)
    d = rsa.make_desc(torch.empty(1, Z, rows, A, device="cuda", dtype=torch.bfloat16), 1)
    X, E, D = rand(1, Z, rows, A), rand(rows, Kp), rand(1, Z, Kp, A)
    Xd, Ed, Dd = X[0].double(), E.double(), D[0].double()
    dX, dE = rsa.linformer_project_bwd(d, D, X, E, dX=X if over else None)
    for z in range(Z):
        close(dX[0, z], Ed @ Dd[z], Ed.abs() @ Dd[z].abs(), Kp)
    x, y = Xd.permute(1, 0, 2).reshape(rows, Z * A), Dd.permute(1, 0, 2).reshape(Kp, Z * A)
    close(dE, x @ y.T, x.abs() @ y.abs().T, Z * A, f32=True)


@pytest.mark.parametrize("rows,Z,A,Kp,chain", [
    (64, 32, 64, 128, 256),
    (2048, 32, 64, 128, 256),
    (2048, 48, 64, 192, 384),
    (1024, 16, 128, 256, 256),
    (16384, 64, 64, 128, 1024),
])
@pytest.mark.parametrize("over", [False, True])
def test_fp32_chains_of_the_projection_matrix_gradient(rows, Z, A, Kp, chain, over):
    """dE sums over all heads in fp32 chains of at most `chain` products, in one grid, in two launches and over X.
    The matrix instruction rounds after every 8 k, each time by 2.5e-8 of the partial sum (RMS: uniform in an ulp, over
    numbers spread evenly by their logarithm), so that a chain of n errs by 2.5e-8 sqrt(n / 16) of its result; the chains'
    own sum errs by 2.5e-8 sqrt(chains / 2).  A quarter more is allowed; chains of twice the length would err by
    1.2 to 1.4 times the model, of four times by 1.6 to 2."""
    torch.manual_seed(rows + Kp)
    d = rsa.make_desc(torch.empty(1, Z, rows, A, device="cuda", dtype=torch.bfloat16), 1)
    X, E, D = rand(1, Z, rows, A), rand(rows, Kp), rand(1, Z, Kp, A)
    x, y = X[0].double().permute(1, 0, 2).reshape(rows, Z * A), D[0].double().permute(1, 0, 2).reshape(Kp, Z * A)
    ref = x @ y.T
    _, dE = rsa.linformer_project_bwd(d, D, X, E, dX=X if over else None)
    err = float((dE.double() - ref).norm() / ref.norm())
    chains = Z * A / chain
    assert err <= 1.25 * 2.53e-8 * (chain / 16 + chains / 2) ** 0.5, err


@pytest.mark.parametrize("rows,Z,H,splits,fold", [(2304, 10, 960, 2, 5), (1344, 13, 832, 3, 5), (2496, 10, 640, 3, 5)])
def test_fp32_chains_of_the_weight_gradient(rows, Z, H, splits, fold):
    """dW in one grid errs no more than by its own launch, which takes more splits at these sizes: as many here, each folded
    after `fold` slabs of 64 rows and added up in turn, with one rounding per 8 rows as the matrix instruction has.  2 % are
    allowed for the difference between that and the instruction."""
    torch.manual_seed(rows)
    d = rsa.make_desc(torch.empty(1, Z, rows, 64, device="cuda", dtype=torch.bfloat16), 1)
    g, X, W = [rand(1, Z, rows, 64) for _ in range(3)], rand(1, rows, H), rand(H, 3 * Z * 64)
    x, y = X[0].double(), torch.cat([heads_to_rows(t) for t in g], 1)
    _, dW = rsa.qkv_proj_bwd(d, *g, X, W)
    ref, total = x.T @ y, None
    per = -(-rows // 64 // splits) * 64
    for s in range(0, rows, per):
        done = None
        for f in range(s, min(s + per, rows), fold * 64):
            acc = torch.zeros_like(dW)
            for k in range(f, min(f + fold * 64, s + per, rows), 8):
                acc = (acc + x[k:k + 8].T @ y[k:k + 8]).float()
            done = acc if done is None else done + acc
        total = done if total is None else total + done
    err, one_launch = (float((t.double() - ref).norm() / ref.norm()) for t in (dW, total))
    print(f"{err:.3e} {one_launch:.3e} {err / one_launch:.3f}")
    assert err <= 1.02 * one_launch
