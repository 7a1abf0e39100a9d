"""The persistent contraction kernels deal the last round of a list, which has fewer tiles than there are CUs, out to all XCDs, unless
that makes the longest walk longer; where contractions are long enough to pay for it, a round of up to a quarter of the CUs goes to
small tiles as a piece of one tensor.  Counts one step off a multiple of the eight XCDs, of a quarter and of a round: short
contractions for the rounds (mostly no piece), longer ones for the pieces, which lomo_contraction_plan confirms.
Every tile has to be computed once: norms against 64 bits (one of 300
tiles is 0.3 % of the sum; fp32 sums over a tile, 2e-5 as in test_gpu_edges.py), stored outputs against 64 bits in full, updates against
the same tensor in two calls."""
import os

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FAMILY = {"norm": "wgrad_sqnorm", "update": "wgrad_update", "dgrad": "dgrad", "forward": "forward", "residual": "forward"}


@pytest.fixture(scope="module")
def L():
    import paper_2306_09782_amd as L
    if not os.path.exists(L.library_path()):
        from paper_2306_09782_amd.build import build
        build(verbose=False)
    L.load_library()
    return L


def normal(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float16)


@pytest.mark.parametrize("tiles", [257, 263, 264, 265, 384, 511, 513, 519])
def test_norm(L, tiles):
    T, K, N = 72, 248, 256 * tiles - 8
    assert L.lomo_contraction_tiles(L.KERNEL_FAMILIES.index("wgrad_sqnorm"), [(T, K, N)]) == [(256, 256)]
    gen = torch.Generator(device=DEV).manual_seed(tiles)
    X, dY = normal(gen, T, K), normal(gen, T, N)
    acc = torch.zeros(1, dtype=torch.float64, device=DEV)
    L.lomo_wgrad_sqnorm(X, dY, acc)
    want = float((dY.double().t().contiguous() @ X.double()).pow(2).sum())
    assert abs(float(acc.item()) / want - 1) < 2e-5


@pytest.mark.parametrize("rows,columns", [(5, 77), (5, 115), (6, 75), (7, 73), (7, 111), (11, 35)])       # of tiles: 385, 575, 450, 511, 777, 385
@pytest.mark.parametrize("product", ["dgrad", "forward", "residual"])
def test_stored(L, rows, columns, product):
    T, M, C = 256 * rows - 8, 256 * columns - 8, 248
    K, N = (M, C) if product == "dgrad" else (C, M)
    assert L.lomo_contraction_plan(L.KERNEL_FAMILIES.index(FAMILY[product]), [(T, K, N)], product == "residual")[0] == [(256, 256)]
    gen = torch.Generator(device=DEV).manual_seed(columns)
    B, W, out, R = normal(gen, T, C), normal(gen, N, K), torch.full((T, M), 7.0, dtype=torch.float16, device=DEV), None
    if product == "residual":
        R = normal(gen, T, M)
        L.lomo_linear_forward_residual(B, W, R, out)
    else:
        (L.lomo_linear_dgrad if product == "dgrad" else L.lomo_linear_forward)(B, W, out)
    b, w = B.double(), W.double() if product == "dgrad" else W.double().t().contiguous()
    want, mag = b @ w, b.abs() @ w.abs()
    if R is not None:
        want, mag = want + R.double(), mag + R.double().abs()
    # fp32 sums of 248 terms: 2^-20 of the sum of their sizes, and half a step of fp16
    assert bool(((out.double() - want).abs() <= 2.0 ** -11 * want.abs() + 2.0 ** -20 * mag).all())


@pytest.mark.parametrize("tiles", [511, 516, 640, 769])
def test_update(L, tiles):
    T, K, N = 1024, 248, 256 * tiles - 8
    assert L.lomo_contraction_tiles(L.KERNEL_FAMILIES.index("wgrad_update"), [(T, K, N)]) == [(256, 256)]
    gen = torch.Generator(device=DEV).manual_seed(tiles)
    X, dY, W = normal(gen, T, K), normal(gen, T, N), normal(gen, N, K)
    whole, half = W.clone(), N // 16 * 8
    L.lomo_linear_backward_update(X, dY, whole, None, 2.0 ** -6, 1.0, 1.0)
    for rows in (slice(0, half), slice(half, N)):
        part = W[rows].clone()
        L.lomo_linear_backward_update(X, dY[:, rows].contiguous(), part, None, 2.0 ** -6, 1.0, 1.0)
        assert torch.equal(part.view(torch.int16), whole[rows].view(torch.int16))


@pytest.mark.parametrize("cut_tensor", ["first", "last"])
def test_piece_of_a_list(L, cut_tensor):
    """16 tiles more than two rounds, in a list: the piece is a row of tiles of the tensor that has sixteen of them side by side."""
    wide, tall = [(4088, 2040)], [(248, 256 * 16 - 8)] * 25      # (K, N): 16 x 8 tiles, 1 x 16 tiles
    shapes = wide + tall if cut_tensor == "first" else tall + wide
    T, gen = 200, torch.Generator(device=DEV).manual_seed(9)
    tensors = [{"kind": "linear", "X": normal(gen, T, K), "dY": normal(gen, T, N), "W": normal(gen, N, K)} for K, N in shapes]
    assert sum(-(-K // 256) * -(-N // 256) for K, N in shapes) == 2 * 256 + 16
    assert set(L.lomo_contraction_tiles(L.KERNEL_FAMILIES.index("wgrad_update"), [(T, K, N) for K, N in shapes])) == {(256, 256)}
    alone, total = [], 0.0
    for t in tensors:
        W, acc = t["W"].clone(), torch.zeros(1, dtype=torch.float64, device=DEV)
        L.lomo_linear_backward_update(t["X"], t["dY"], W, None, 2.0 ** -6, 1.0, 1.0)
        L.lomo_wgrad_sqnorm(t["X"], t["dY"], acc)
        alone.append(W)
        total += float(acc.item())
    lst = L.make_tensor_list(tensors)
    ws = torch.empty(max(256, L.lomo_step_workspace_bytes(lst)), dtype=torch.uint8, device=DEV)
    acc, flags = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(len(shapes) + 1, dtype=torch.int32, device=DEV)
    L.lomo_step_norm_pass(lst, acc, flags, ws)
    assert abs(float(acc.item()) / total - 1) < 1e-6 and not flags.any()
    L.lomo_step_update_pass(lst, 2.0 ** -6, 1.0, 1.0, flags[-1:], ws)
    for t, W in zip(tensors, alone):
        assert torch.equal(t["W"].view(torch.int16), W.view(torch.int16))


# tiles of rows and columns, ragged ends; the piece that is cut: two columns of tiles, or one row
@pytest.mark.parametrize("rows,columns,piece", [(5, 53, (504, 1272)), (52, 5, (1272, 248))])
@pytest.mark.parametrize("product", sorted(FAMILY))
def test_piece(L, rows, columns, piece, product):
    n, m, C = 256 * rows - 8, 256 * columns - 8, 1032
    T, K, N = {"dgrad": (n, m, C), "forward": (n, C, m), "residual": (n, C, m)}.get(product, (C, m, n))
    tiles, (tensor, cut, small, _) = L.lomo_contraction_plan(L.KERNEL_FAMILIES.index(FAMILY[product]), [(T, K, N)], product == "residual")
    assert tiles == [(256, 256)] and tensor == 0 and cut == piece and small != (256, 256)
    gen = torch.Generator(device=DEV).manual_seed(rows)
    if product in ("norm", "update"):
        X, dY = normal(gen, T, K), normal(gen, T, N)
        G = dY.double().t().contiguous() @ X.double()
        if product == "norm":
            acc, flag = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
            L.lomo_wgrad_sqnorm(X, dY, acc, flag)
            assert abs(float(acc.item()) / float(G.pow(2).sum()) - 1) < 2e-5 and int(flag.item()) == 0
            # an element of the piece alone raises the flag
            (dY if cut[1] < cut[0] else X)[3, -1] = float("inf")
            L.lomo_wgrad_sqnorm(X, dY, acc, flag)
            assert int(flag.item()) == 1
        else:
            W = normal(gen, N, K)
            whole, half = W.clone(), N // 16 * 8
            L.lomo_linear_backward_update(X, dY, whole, None, 2.0 ** -6, 1.0, 1.0)
            for part in (slice(0, half), slice(half, N)):
                one = W[part].clone()
                L.lomo_linear_backward_update(X, dY[:, part].contiguous(), one, None, 2.0 ** -6, 1.0, 1.0)
                assert torch.equal(one.view(torch.int16), whole[part].view(torch.int16))
            want = W.double() - 2.0 ** -6 * G
            assert bool(((whole.double() - want).abs() <= 2.0 ** -11 * want.abs() + 2.0 ** -20 * 2.0 ** -6 * T * 8).all())
        return
    B, W, out, R = normal(gen, T, C), normal(gen, N, K), torch.full((T, m), 7.0, dtype=torch.float16, device=DEV), None
    if product == "residual":
        R = normal(gen, T, m)
        L.lomo_linear_forward_residual(B, W, R, out)
    else:
        (L.lomo_linear_dgrad if product == "dgrad" else L.lomo_linear_forward)(B, W, out)
    b, w = B.double(), W.double() if product == "dgrad" else W.double().t().contiguous()
    want, mag = b @ w, b.abs() @ w.abs()
    if R is not None:
        want, mag = want + R.double(), mag + R.double().abs()
    assert bool(((out.double() - want).abs() <= 2.0 ** -11 * want.abs() + 2.0 ** -20 * mag).all())


@pytest.mark.parametrize("order", ["dealt out", "left to the first XCDs"])
def test_last_round_of_a_list_of_different_contractions(L, order):
    """96 tiles in the last round: where the first XCDs' workgroups have had short contractions in every round, and dealt out some would
    come on top of long ones, they stay with the first."""
    short, long_ = (2560, 1032), (1536, 2056)      # (K, N) of dX: 160 tiles and 96
    shapes = [short, long_] * 2 + [(1536, 1032)] if order != "dealt out" else [long_, short] * 2 + [(1536, 1032)]
    T, gen = 4088, torch.Generator(device=DEV).manual_seed(2)
    tiles, (tensor, _, _, dealt) = L.lomo_contraction_plan(L.KERNEL_FAMILIES.index("dgrad"), [(T, K, N) for K, N in shapes])
    assert set(tiles) == {(256, 256)} and tensor is None and dealt == (order == "dealt out")
    tensors = [{"kind": "linear", "X": torch.zeros(T, K, dtype=torch.float16, device=DEV), "dY": normal(gen, T, N), "W": normal(gen, N, K),
                "dX": torch.full((T, K), 7.0, dtype=torch.float16, device=DEV)} for K, N in shapes]
    lst = L.make_tensor_list(tensors)
    ws = torch.empty(max(256, L.lomo_step_workspace_bytes(lst)), dtype=torch.uint8, device=DEV)
    L.lomo_step_update_pass(lst, 2.0 ** -6, 1.0, 1.0, torch.zeros(1, dtype=torch.int32, device=DEV), ws)      # X is zero: W stays
    for t in tensors:
        alone = torch.empty_like(t["dX"])
        L.lomo_linear_dgrad(t["dY"], t["W"], alone)
        assert torch.equal(alone.view(torch.int16), t["dX"].view(torch.int16))
