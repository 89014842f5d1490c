"""Which kernels a call takes, on the CPU: the cases of the GPU tests of a dispatch reach the forms that they are there for."""
import ctypes
import random

import pytest

import launches
import test_gpu_backward_one_grid as one_grid
import test_gpu_gradients_one_grid as gradients
import test_gpu_projected_keys_backward as projected
import test_gpu_projection_in_one_split as one_split
import test_gpu_staged as staged
import test_gpu_staged_by_keys as by_keys
import test_gpu_staged_groups as groups
import test_gpu_staged_one_pass as one_pass
from paper_2105_13120_amd import rsa


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    return launches.Recorder(str(tmp_path_factory.mktemp("recorder")))


def params(test, name=None):
    """The parameters of a test's only (or of its `name`) parametrisation."""
    marks = [m for m in test.pytestmark if m.name == "parametrize" and (name is None or m.args[0] == name)]
    return marks[-1].args[1]


def names(calls):
    return [k.name for k in calls]


# fused_bwd_both_kernel's shape by (halves of a head, groups of waves on a walk)
BOTH = {(1, 4): "1, 1, 1, 4, 1, 1, 4", (1, 2): "1, 1, 2, 2, 1, 2, 2", (1, 1): "1, 2, 4, 1, 2, 4, 1",
        (2, 2): "2, 1, 2, 2, 1, 2, 2", (2, 1): "2, 2, 4, 1, 1, 4, 1"}


@pytest.mark.parametrize("case,on_a_walk", zip(one_grid.CASES, [4, 4, 4, 2, 2, 2, 1, 1, 1, 2, 4, 2, 1, 1]))
def test_backward_in_one_grid(rec, case, on_a_walk):
    A, B, Z, L, N, rb, re, causal, zigzag = case
    d = launches.descriptor(B, Z, L, N, A, (rb, re), causal, zigzag)
    both = f"fused_bwd_both_kernel<{str(causal).lower()}, {BOTH[A // 64, on_a_walk]}>"
    assert names(launches.backward(rec, d)) == ["bwd_preprocess_kernel", both]
    assert names(rec("bwd_dkdv", d, "dO", "Q", "K", "V", "ws", "dK", "dV"))[0].startswith("fused_bwd_dkdv_kernel")
    assert names(rec("bwd_dq", d, "dO", "Q", "K", "V", "ws", "dQ"))[0].startswith("fused_bwd_dq_kernel")


@pytest.mark.parametrize("case,one", zip(params(one_grid.test_gradients_over_keys_and_values, "A,B,Z,L,N,causal"), [True, True, True, False]))
def test_backward_over_keys_and_values_takes_two_grids(rec, case, one):
    A, B, Z, L, N, causal = case
    d = launches.descriptor(B, Z, L, N, A, causal=causal)
    assert any("both" in n for n in names(launches.backward(rec, d))) == one
    for dK, dV in (("K", "V"), ("V", "K"), ("K", "dV"), ("dK", "K")):
        assert not any("both" in n for n in names(launches.backward(rec, d, dK, dV)))


# groups of waves: fp32 forward in one pass (0: the strip), fp32 apply, collect, bf16 apply, collect
STAGED = [(4, 4, 4, 4, 1), (4, 4, 4, 4, 1), (0, 4, 4, 4, 2), (2, 2, 2, 2, 1), (2, 2, 2, 4, 1), (4, 2, 2, 4, 2), (0, 2, 2, 2, 2),
          (1, 2, 2, 2, 1), (2, 1, 1, 1, 1), (1, 1, 1, 1, 1), (2, 2, 2, 2, 1), (4, 4, 2, 4, 1), (2, 1, 1, 2, 1), (0, 2, 2, 2, 1)]


@pytest.mark.parametrize("case,on_a_walk", zip(groups.CASES, STAGED))
def test_two_pass_groups(rec, case, on_a_walk):
    B, Z, L, N, A, rb, re, causal = case

    def last(kernels, start):  # (the last number of a kernel's shape: its groups)
        return [int(n.rstrip(">").split(", ")[-1]) for n in names(kernels) if n.startswith(start)]

    one_pass, *rest = on_a_walk
    for dtype, apply, collect in ((rsa.RSA_F32, *rest[:2]), (rsa.RSA_BF16, *rest[2:])):
        d = launches.descriptor(B, Z, L, N, A, (rb, re), causal, dtype=dtype, mode=rsa.MODE_STAGED)
        fwd, bwd = launches.forward(rec, d), launches.backward(rec, d)
        assert last(bwd, "strip_apply") == [apply] and last(bwd, "strip_collect") == [collect]
        assert last(fwd, "f32_forward") == ([one_pass] if dtype == rsa.RSA_F32 and one_pass else [])


@pytest.mark.parametrize("case,one_step", groups.STEP_CASES)
def test_two_pass_fp32_walks_of_one_step(rec, case, one_step):
    B, Z, L, N, A, rb, re, causal = case
    d = launches.descriptor(B, Z, L, N, A, (rb, re), causal, dtype=rsa.RSA_F32, mode=rsa.MODE_STAGED)
    assert names(launches.forward(rec, d)) == [("f32_forward_step_kernel" if one_step else "f32_forward_kernel") + "<1, 4>"]


@pytest.mark.parametrize("case", params(staged.test_f32_one_pass_on_long_walks, "B,Z,L,N,causal,on_a_walk"))
def test_two_pass_long_walks_in_one_pass(rec, case):
    B, Z, L, N, causal, on_a_walk = case
    d = launches.descriptor(B, Z, L, N, causal=causal, dtype=rsa.RSA_F32, mode=rsa.MODE_STAGED)
    assert names(launches.forward(rec, d)) == [f"f32_forward_kernel<{4 // on_a_walk}, {on_a_walk}>"]


@pytest.mark.parametrize("case,strip", one_pass.CASES)
def test_two_pass_forward_keeps_a_strip_where_rows_are_few(rec, case, strip):
    B, Z, L, N, A, rb, re, causal = case
    d = launches.descriptor(B, Z, L, N, A, (rb, re), causal, mode=rsa.MODE_STAGED)
    got = names(launches.forward(rec, d))
    assert [n.startswith("strip_scores_fwd") for n in got] == [True, False] if strip else [n.startswith("fused_fwd") for n in got] == [True]


# heads, L, N, ranks, causal; rows a wave, waves on the rows, groups of waves
@pytest.mark.parametrize("heads,L,N,ranks,causal,shape,grid", [
    (1, 16384, 1, (0, 1), False, (32, 2, 4), 256),
    (1, 16384, 1, (0, 1), True, (32, 2, 4), 256),
    (4, 8192, 1, (0, 1), False, (32, 4, 2), 256),
    (16, 16384, 16, (3, 4), False, (32, 2, 4), 256),
    (130, 4096, 8, (5, 6), False, (32, 4, 1), 520),
    (64, 8192, 8, (4, 5), False, (64, 4, 1), 256),
    (256, 4096, 8, (7, 8), True, (64, 4, 1), 512),
])
def test_walks_without_room_for_a_split_are_not_planned_with_one(rec, heads, L, N, ranks, causal, shape, grid):
    d = launches.descriptor(1, heads, L, N, 64, ranks, causal, mode=rsa.MODE_STAGED)
    (k,) = launches.forward(rec, d)
    rows, waves, on_a_walk = shape
    assert k.name == f"fused_fwd_kernel<{rows}, {str(causal).lower()}, 1, {rows // 32}, {waves}, {on_a_walk}, true>"
    assert k.grid == (grid, 1, 1)


# heads of 128: on either side of the lines
@pytest.mark.parametrize("heads,L,N,ranks,causal,one_pass", [
    (2, 4608, 1, (0, 1), False, False), (4, 4608, 1, (0, 1), False, True), (16, 640, 1, (0, 1), False, True),
    (5, 1600, 1, (0, 1), True, False), (10, 1600, 1, (0, 1), True, True),                  # whole causal rings
    (2, 8192, 1, (0, 1), True, False), (3, 8192, 1, (0, 1), True, True),
    (8, 5120, 4, (2, 3), True, False), (14, 5120, 4, (2, 3), True, True),                  # walks about as long
    (66, 8192, 128, (0, 1), True, True), (80, 320, 5, (4, 5), False, True),                # few keys
])
def test_two_pass_forward_of_heads_of_128(rec, heads, L, N, ranks, causal, one_pass):
    got = names(launches.forward(rec, launches.descriptor(1, heads, L, N, 128, ranks, causal, mode=rsa.MODE_STAGED)))
    assert any(n.startswith("fused_fwd_kernel") for n in got) == one_pass


# the shape: waves along the rows, groups of waves on a walk
@pytest.mark.parametrize("heads,L,N,A,ranks,shape", [
    (300, 1024, 16, 64, (0, 1), "4, 1"), (300, 1024, 16, 128, (0, 1), "4, 1"), (75, 2048, 4, 64, (0, 1), "4, 1"),  # few keys
    (18, 8192, 4, 64, (0, 1), "2, 4"), (264, 1024, 16, 128, (0, 1), "4, 1"),
    (264, 1024, 16, 128, (15, 16), "4, 1"), (420, 1024, 16, 128, (8, 9), "4, 1"), (256, 1024, 16, 128, (15, 16), "4, 2"),  # walks as long
    (38, 2048, 4, 128, (0, 2), "4, 2"), (33, 1024, 1, 128, (0, 1), "4, 2"),                                               # and others
])
def test_two_pass_shapes_go_by_what_the_rows_see(rec, heads, L, N, A, ranks, shape):
    (k,) = launches.forward(rec, launches.descriptor(1, heads, L, N, A, ranks, True, mode=rsa.MODE_STAGED))
    assert k.name == f"fused_fwd_kernel<32, true, {A // 64}, 1, {shape}, true>"


# rows of one rank's share that are no multiple of 256; rows of a work-group
@pytest.mark.parametrize("heads,L,N,ranks,causal,rows", [
    (202, 2944, 2, (1, 2), False, 256),    # as many rounds of large work-groups as of two small ones in their place,
    (260, 1344, 3, (2, 3), False, 128),    # one more
    (200, 2112, 3, (2, 3), False, 128),
    (200, 1408, 2, (1, 2), True, 128),
    (202, 2944, 2, (1, 2), True, 128),
])
def test_forward_of_a_ragged_share(rec, heads, L, N, ranks, causal, rows):
    (k,) = launches.forward(rec, launches.descriptor(1, heads, L, N, 64, ranks, causal))
    assert k.grid == (heads * -(-(L // N) // rows), 1, 1)


@pytest.mark.parametrize("heads,rows,Kp,want", [(192, 960, 1024, 256), (64, 960, 1024, 128), (128, 448, 2048, 128), (137, 960, 1024, 128), (192, 960, 512, 128), (260, 448, 512, 128)])
def test_ragged_rows_to_projected_keys(rec, heads, rows, Kp, want):
    (k,) = rec("linformer_forward", launches.descriptor(1, heads, rows, 1), Kp, "Q", "K", "V", "O", "LSE")
    assert k.grid == (heads * -(-rows // want), 1, 1)


@pytest.mark.parametrize("heads,rows,grid", [(160, 512, 640), (48, 2560, 480)])
def test_attention_to_many_projected_keys_fills_the_chip(rec, heads, rows, grid):
    (k,) = rec("linformer_forward", launches.descriptor(1, heads, rows, 1), 4096, "Q", "K", "V", "O", "LSE")
    assert k.grid == (grid, 1, 1)


# groups of waves of the kernel that walks the rows, and groups of heads
@pytest.mark.parametrize("case,on_a_walk,of_heads", zip(by_keys.CASES, [1, 1, 1, 1, 2, 4, 1, 1, 2, 1, 1, 2, 1], [1] * 10 + [3, 3, 3]))
def test_two_pass_backward_by_keys(rec, case, on_a_walk, of_heads):
    B, Z, L, N, A, rb, re, causal = case
    d = launches.descriptor(B, Z, L, N, A, (rb, re), causal, mode=rsa.MODE_STAGED)
    first, *rest = names(launches.backward(rec, d))
    assert first == "bwd_preprocess_kernel" and len(rest) == 2 * of_heads
    shape = {1: "4, 1", 2: "2, 2", 4: "2, 4"}[on_a_walk]
    assert set(rest[::2]) == {f"strip_collect_keys_kernel<{str(causal).lower()}, {A // 64}, {shape}>"}
    assert all(n.startswith("strip_apply_keys") for n in rest[1::2])


@pytest.mark.parametrize("case", by_keys.BY_ROWS)
def test_two_pass_backward_by_rows_near_the_line(rec, case):
    B, Z, L, N, A, rb, re, causal = case
    d = launches.descriptor(B, Z, L, N, A, (rb, re), causal, mode=rsa.MODE_STAGED)
    assert not any(n.startswith("strip_collect_keys") for n in names(launches.backward(rec, d)))


# heads, L, N, A, ranks, causal: on either side of the lines
@pytest.mark.parametrize("heads,L,N,A,ranks,causal,by_keys", [
    (9, 2048, 4, 64, (0, 1), False, False), (16, 2048, 4, 64, (0, 1), False, True),      # work-groups that dQ has
    (9, 2048, 4, 64, (3, 4), True, False), (16, 2048, 4, 64, (3, 4), True, True),
    (75, 512, 8, 64, (7, 8), True, False), (130, 512, 8, 64, (7, 8), True, True),        # one tile of rows
    (200, 1024, 16, 64, (0, 1), True, False), (200, 1024, 16, 64, (8, 9), True, True),   # keys that no row sees
    (256, 64, 1, 128, (0, 1), False, False), (128, 256, 1, 128, (0, 1), False, True),    # heads of 128: rounds of one work-group to a CU
    (150, 256, 1, 128, (0, 1), False, False), (100, 512, 1, 128, (0, 1), False, True),
    (85, 320, 1, 128, (0, 1), True, False), (41, 768, 1, 128, (0, 1), True, False), (32, 1024, 1, 128, (0, 1), True, True),
    (100, 448, 1, 128, (0, 1), True, True), (62, 512, 8, 128, (7, 8), True, False),
    (125, 1024, 8, 128, (7, 8), True, False), (65, 1024, 2, 128, (1, 2), True, True),
    (9, 3968, 2, 128, (0, 1), True, False), (16, 3968, 2, 128, (0, 1), True, True),      # ... that see some rows
    (121, 2240, 5, 128, (0, 1), True, False), (121, 2240, 5, 128, (1, 2), True, True),
    (21, 1792, 1, 128, (0, 1), False, True), (12, 3584, 4, 128, (3, 4), True, False), (22, 4096, 4, 128, (3, 4), True, True),
])
def test_two_pass_backward_takes_the_faster_way(rec, heads, L, N, A, ranks, causal, by_keys):
    got = names(launches.backward(rec, launches.descriptor(1, heads, L, N, A, ranks, causal, mode=rsa.MODE_STAGED)))
    assert any(n.startswith("strip_collect_keys") for n in got) == by_keys


def shifted_backward(rec, d):
    """Status of a two-pass backward whose dK starts at the 65th row of K, with the workspace that every call is asked for."""
    at = lambda i: (i + 1) << 40
    ws = rec.lib.rsa_workspace_bytes(ctypes.byref(d), 1)
    return rec.lib.rsa_backward(ctypes.byref(d), at(0), at(1), at(2), at(3), at(4), at(5), at(6), at(2) + 64 * d.A * 2, at(7), at(8), ws, None), ws


# (accepted with the strips by rows, whose least plan holds 128 rows of a head)
@pytest.mark.parametrize("heads,L,N,A,causal", [(126, 3200, 10, 64, False), (101, 2496, 3, 128, True)])
def test_backward_by_keys_where_results_fill_the_workspace(rec, heads, L, N, A, causal):
    assert shifted_backward(rec, launches.descriptor(1, heads, L, N, A, None, causal, mode=rsa.MODE_STAGED))[0] == 0


def test_two_pass_backward_over_its_inputs_needs_no_more_than_by_rows(rec):
    """Wherever all results and the strips of 128 rows of a head fit what every call is asked for, results may lie over inputs in
    any way, also by keys, whose strip is a whole head's."""
    rng = random.Random(5)
    up = lambda n: (n + 255) // 256 * 256
    told = 0
    for _ in range(4000):
        N = rng.randint(1, 8)
        c = 64 * rng.randint(1, max(1, 64 // N))
        rb = rng.randrange(N)
        re = rng.randint(rb + 1, N) if rng.random() < 0.3 else N
        d = launches.descriptor(1, rng.randint(1, 200), N * c, N, rng.choice([64, 128]), (rb, re), rng.random() < 0.5, mode=rsa.MODE_STAGED)
        Lq = (re - rb) * c
        rows = min(Lq, 128)
        need = up(d.Z * Lq * d.A * 2) + 2 * up(d.Z * d.L * d.A * 2) + 2 * up(rows * d.L * 2) + (2 * up(d.L * d.A * 4) if rows < Lq else 0)
        status, ws = shifted_backward(rec, d)
        if need <= ws:
            told += 1
            assert status == 0, (d.Z, d.L, d.N, d.A, rb, re, d.causal)
    assert told > 1000


def tiles(launch):
    """(T, groups) of the products of a launch."""
    t = [x.strip() for x in launch.name[launch.name.index("<") + 1:-1].split(",")]
    if launch.name.startswith("proj_gemm_pair"):
        return (int(t[2]), int(t[3])), (int(t[4]), int(t[5]))
    return ((int(t[4]), int(t[5])),)


# the input's and the weights' gradient, in one grid or (None) in two: of the Q/K/V map, of the output map
SMALL, LARGE = (1, 2), (4, 1)
MAPS = [((SMALL, SMALL), (SMALL, SMALL)), ((SMALL, SMALL), (SMALL, SMALL)), ((SMALL, SMALL), (SMALL, SMALL)),
        (None, ((2, 1), (2, 1))), (((2, 1), (2, 1)), ((2, 1), SMALL)), (None, ((2, 1), (2, 1))),
        (((2, 1), (2, 1)), ((2, 1), (2, 1))), (None, (LARGE, (2, 2))),
        ((SMALL, (2, 1)), (SMALL, (2, 1))), ((LARGE, (2, 2)), (SMALL, SMALL)), ((LARGE, LARGE), (LARGE, (2, 2))),
        ((LARGE, LARGE), ((2, 1), (2, 1)))]


@pytest.mark.parametrize("case,want", zip(params(gradients.test_maps), MAPS))
def test_gradients_of_the_maps(rec, case, want):
    rows, Z, A, H = case
    d = launches.descriptor(1, Z, rows, 1, A)
    for call, form in zip((rec("qkv_proj_bwd", d, H, "dQ", "dK", "dV", "X", "W", "dX", "dW", "ws"),
                           rec("out_proj_bwd", d, H, "dY", "O", "Wo", "dO", "dWo", "ws")), want):
        got = [tiles(k) for k in call if k.name.startswith("proj_gemm")]
        if form:
            assert got == [form]
        else:
            assert len(got) == 2
    # dW over W keeps two launches
    assert len([k for k in rec("qkv_proj_bwd", d, H, "dQ", "dK", "dV", "X", "W", "dX", "W", "ws") if "gemm" in k.name]) == 2


ALONG = [(SMALL, SMALL), (SMALL, SMALL), ((2, 1), SMALL), ((2, 1), (2, 1)), ((2, 1), (2, 1)), ((2, 1), (2, 1)), None, (LARGE, LARGE),
         (LARGE, LARGE), ((2, 1), (2, 1))]


@pytest.mark.parametrize("case,want", zip(params(gradients.test_projection_along_the_sequence), ALONG))
def test_gradients_of_the_projection_along_the_sequence(rec, case, want):
    rows, Z, A, Kp, over = case
    d = launches.descriptor(1, Z, rows, 1, A)
    got = [tiles(k) for k in rec("linformer_project_bwd", d, Kp, "dXp", "X", "E", "X" if over else "dX", "dE") if "gemm" in k.name]
    assert got == [want] if want else len(got) == 2


@pytest.mark.parametrize("case,form", one_split.CASES)
def test_projection_along_the_sequence_in_one_split(rec, case, form):
    heads, L, N, rb, re, Kp, A = case
    d = launches.descriptor(1, heads, L, N, A, (rb, re))
    got = rec("linformer_project", d, Kp, "X", "E", "Xp", "ws")
    assert len(got) == 1 and tiles(got[0]) == (form,) and got[0].name.startswith("proj_gemm_kernel<true, true, false")
    assert names(rec("linformer_project", d, Kp, "X", "E", "X", "ws"))[1:] == ["ksplit_reduce_heads_kernel"]


@pytest.mark.parametrize("rows,Z,A,Kp", [(16384, 64, 64, 128), (80640, 22, 128, 128)])
def test_gradients_that_are_bound_by_memory_take_two_launches(rec, rows, Z, A, Kp):
    kernels = names(rec("linformer_project_bwd", launches.descriptor(1, Z, rows, 1, A), Kp, "dXp", "X", "E", "dX", "dE"))
    assert any(k.startswith("linformer_dx") for k in kernels) and not any(k.startswith("proj_gemm_pair") for k in kernels)


# blocks of 32 keys, groups, splits
@pytest.mark.parametrize("case,want", zip(params(projected.test_few_keys), [
    (1, 4, 8), (1, 4, 16), (1, 4, 1), (4, 1, 4), (2, 2, 8), (1, 4, 8), (2, 2, 8), (2, 2, 1)]))
def test_few_projected_keys(rec, case, want):
    B, Z, L, N, ranks, Kp, A = case
    d = launches.descriptor(B, Z, L, N, A, ranks)
    kernels = rec("linformer_backward", d, Kp, "dO", "Q", "Kp", "Vp", "O", "LSE", "dQ", "dKp", "dVp", "ws")
    k = next(k for k in kernels if k.name.startswith("fused_bwd_dkdv"))
    assert (*(int(x) for x in k.name.rstrip(">").split(", ")[-2:]), k.grid[1]) == want
    assert any(k.name.startswith("qsplit_reduce") for k in kernels) == (want[2] > 1)
