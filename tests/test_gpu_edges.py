"""The contraction kernels at the edges of their tiles and slices: sizes one step off a whole tile (256 and 128) or a
whole slice (32 and 64 contraction indices), the smallest sizes, and a non-finite neighbour just outside a short slice.

Bars as in test_gpu_parity.py: W within 1 fp16 ulp on 99.9 %, 2 everywhere; dX and Y also within 2^-20 of the sum of the
absolute products where the sum cancels (fp32 sums of at most 2^12 terms); the norm within 2e-5; flags exact.  Every
output lies in a larger buffer whose other elements must keep their bits."""
import math
import os

import numpy as np
import pytest
import torch

import lomo_synth as S
from oracle import lomo_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PAD = 512          # guarded elements on either side of an output


@pytest.fixture(scope="module")
def L():
    import paper_2306_09782_amd as L
    if not os.path.exists(L.library_path()):
        from paper_2306_09782_amd.build import build
        build(verbose=False)
    L.load_library()
    return L


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def f16(seed, shape, sigma, scale=1.0):
    return S.normal_f16_np(S.tensor_key(81, seed, shape[0], shape[1]), shape, S.normal_mult(sigma, scale))


class Guarded:
    """A device tensor inside a larger buffer of sevens."""

    def __init__(self, shape, init=None):
        n = shape[0] * shape[1]
        self.whole = torch.full((n + 2 * PAD,), 7.0, dtype=torch.float16, device=DEV)
        self.t = self.whole[PAD:PAD + n].view(shape)
        if init is not None:
            self.t.copy_(dev(init))

    def host(self):
        w = self.whole.cpu().numpy()
        assert (w[:PAD] == 7).all() and (w[-PAD:] == 7).all(), "written outside the output"
        return self.t.cpu().numpy()


def product_ok(got, ref64, mag, what):
    d = O.ulp_distance_f16(got, O.round_f16(ref64))
    near = np.abs(got.astype(np.float64) - ref64) <= 2.0 ** -20 * mag
    assert ((d <= 2) | near).all(), f"{what}: off by {d.max()} ulp"
    assert ((d <= 1) | near).mean() >= 0.999, what


def weights_ok(got, want, what):
    d = O.ulp_distance_f16(got, want)
    assert d.max() <= 2 and (d <= 1).mean() >= 0.999, (what, int(d.max()))


SHAPES = [(1, 8, 8), (7, 8, 264), (31, 264, 8), (32, 256, 256), (33, 248, 520), (63, 136, 128), (65, 120, 384), (96, 384, 136),
          (127, 256, 776), (128, 512, 512), (129, 264, 248), (255, 1032, 72), (257, 72, 1032), (260, 520, 2056), (777, 504, 504)]


@pytest.mark.parametrize("T,K,N", SHAPES)
def test_step_at_tile_and_slice_edges(L, T, K, N):
    step_matches_oracle(L, T, K, N)


# Ragged shapes for each kernel a tensor can go to, and a contraction of one index with many tiles
TILES = {(777, 1544, 1032): ((128, 64), (128, 64), (128, 64)), (300, 3080, 4104): ((256, 256), (64, 64), (256, 256)),
         (3080, 3336, 3848): ((256, 256), (256, 256), (256, 256)), (904, 1160, 2056): ((128, 128), (128, 64), (128, 128)),
         (1016, 2056, 3080): ((128, 128), (128, 128), (128, 128)), (1, 2056, 4104): ((128, 64), (64, 64), (256, 256)),
         (777, 504, 504): ((64, 64), (64, 64), (64, 64))}


@pytest.mark.parametrize("T,K,N", TILES)
def test_step_in_each_tile_shape(L, T, K, N):
    got = [L.lomo_contraction_tiles(L.KERNEL_FAMILIES.index(f), [(T, K, N)])[0] for f in ("wgrad_update", "dgrad", "wgrad_sqnorm")]
    assert tuple(got) == TILES[T, K, N], "this shape no longer exercises the kernels it is here for: choose another"
    step_matches_oracle(L, T, K, N)


@pytest.mark.parametrize("T", [129, 600])
def test_lists_of_unequal_tensors(L, T):
    """More tensors than one launch's table holds, contraction lengths from 8 to 4104: each result has the bits it has alone."""
    shapes = [(264, 8), (8, 4104), (520, 1032)] * 15
    tensors, alone = [], []
    for i, (K, N) in enumerate(shapes):
        X, dY, W = f16(20 + i, (T, K), 1.0), f16(90 + i, (T, N), 1.0), f16(160 + i, (N, K), 0.02)
        tensors.append({"kind": "linear", "X": dev(X), "dY": dev(dY), "W": dev(W), "dX": torch.zeros(T, K, dtype=torch.float16, device=DEV)})
        dX, W2 = torch.empty(T, K, dtype=torch.float16, device=DEV), dev(W)
        L.lomo_linear_backward_update(tensors[-1]["X"], tensors[-1]["dY"], W2, dX, 1e-3, 1.0, 1.0)
        alone.append((W2, dX))
    lst = L.make_tensor_list(tensors)
    ws = torch.empty(max(256, L.lomo_step_workspace_bytes(lst)), dtype=torch.uint8, device=DEV)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    L.lomo_step_update_pass(lst, 1e-3, 1.0, 1.0, flag, ws)
    for i, (t, (W2, dX)) in enumerate(zip(tensors, alone)):
        assert torch.equal(t["W"], W2) and torch.equal(t["dX"], dX), i
        d64, w64 = t["dY"].cpu().numpy().astype(np.float64), f16(160 + i, shapes[i][::-1], 0.02).astype(np.float64)
        product_ok(dX.cpu().numpy(), d64 @ w64, np.abs(d64) @ np.abs(w64), f"dX {i}")


def test_a_list_takes_other_tiles_than_its_tensors_alone(L):
    """Whole-tile tensors that alone are cut into small tiles share the persistent kernel in a list, the long contraction
    excepted: same bits, and the list's norm is the sum of the norms."""
    shapes = [(512, 1024, 1024), (512, 2816, 1024)] * 30 + [(512, 1024, 32000)]
    fam = {k: L.KERNEL_FAMILIES.index(k) for k in ("dgrad", "wgrad_update", "wgrad_sqnorm")}
    for f in fam.values():
        together, alone = L.lomo_contraction_tiles(f, shapes), [L.lomo_contraction_tiles(f, [s])[0] for s in shapes]
        assert together[0] == (256, 256) and alone[0] != (256, 256)
    assert L.lomo_contraction_tiles(fam["dgrad"], shapes)[-1] != (256, 256)
    tensors, alone, total = [], [], 0.0
    gen = torch.Generator(device=DEV).manual_seed(5)
    normal = lambda shape, sigma: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float16) * sigma
    for T, K, N in shapes:
        t = {"kind": "linear", "X": normal((T, K), 1.0), "dY": normal((T, N), 1.0), "W": normal((N, K), 0.02),
             "dX": torch.zeros(T, K, dtype=torch.float16, device=DEV)}
        tensors.append(t)
        dX, W2, acc = torch.empty_like(t["dX"]), t["W"].clone(), torch.zeros(1, dtype=torch.float64, device=DEV)
        L.lomo_wgrad_sqnorm(t["X"], t["dY"], acc)
        L.lomo_linear_backward_update(t["X"], t["dY"], W2, dX, 1e-3, 1.0, 1.0)
        total += float(acc.item())
        alone.append((W2, dX))
    lst = L.make_tensor_list(tensors)
    ws = torch.empty(max(256, L.lomo_step_workspace_bytes(lst)), dtype=torch.uint8, device=DEV)
    acc, flags = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(len(shapes) + 1, dtype=torch.int32, device=DEV)
    L.lomo_step_norm_pass(lst, acc, flags, ws)
    assert abs(float(acc.item()) / total - 1) < 1e-6 and not flags.any()          # fp32 sums over a tile, fp64 over tiles
    L.lomo_step_update_pass(lst, 1e-3, 1.0, 1.0, flags[-1:], ws)
    for i, (t, (W2, dX)) in enumerate(zip(tensors, alone)):
        assert torch.equal(t["W"].view(torch.int16), W2.view(torch.int16)) and torch.equal(t["dX"].view(torch.int16), dX.view(torch.int16)), i


def step_matches_oracle(L, T, K, N):
    """Norm, visible update, dX and the clip-by-value update through the whole-pass calls."""
    Sc = 256.0
    X, dY, W = f16(1, (T, K), 1.0), f16(2, (T, N), 0.01, Sc), f16(3, (N, K), 0.02)
    G = O.linear_grad(X, dY)
    Wd, dX = Guarded((N, K), W), Guarded((T, K))
    tensor = {"kind": "linear", "X": dev(X), "dY": dev(dY), "W": Wd.t, "dX": dX.t}
    lst = L.make_tensor_list([tensor])          # holds addresses: `tensor` keeps them alive
    ws = torch.empty(max(256, L.lomo_step_workspace_bytes(lst)), dtype=torch.uint8, device=DEV)
    acc, flags = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(2, dtype=torch.int32, device=DEV)
    L.lomo_step_norm_pass(lst, acc, flags, ws)
    assert abs(float(acc.item()) / O.sqnorm(G) - 1) < 2e-5 and flags.cpu().tolist() == [0, 0]
    lr = float(np.float32(30 * 2.0 ** -16 / (math.sqrt(T) * 0.01)))
    L.lomo_step_update_pass(lst, lr, 1.0 / Sc, 1.0, flags[1:], ws)
    weights_ok(Wd.host(), O.sgd_update(W, G, lr, 1.0, Sc), "W")
    a64 = dY.astype(np.float64), W.astype(np.float64)
    product_ok(dX.host(), a64[0] @ a64[1], np.abs(a64[0]) @ np.abs(a64[1]), "dX")
    Wd.t.copy_(dev(W))
    clipv = float(np.float32(0.005 * math.sqrt(T)))          # clips about half of the elements
    L.lomo_step_update_pass_clip_value(lst, 0.02, 1.0 / Sc, clipv, flags, ws)
    weights_ok(Wd.host(), O.sgd_update_clip_value(W, G, float(np.float32(0.02)), clipv, Sc), "W by value")
    assert flags.cpu().tolist() == [0, 0]


@pytest.mark.parametrize("T,K,N", [(1, 8, 8), (33, 40, 264), (64, 264, 136), (127, 72, 384), (129, 520, 248), (257, 1032, 520),
                                   (4100, 40, 3080), (3080, 104, 4104)])
@pytest.mark.parametrize("residual", [False, True])
def test_forward_at_tile_and_slice_edges(L, T, K, N, residual):
    X, W, R = f16(4, (T, K), 1.0), f16(5, (N, K), 0.05), f16(6, (T, N), 1.0)
    Y = Guarded((T, N))
    if residual:
        L.lomo_linear_forward_residual(dev(X), dev(W), dev(R), Y.t)
    else:
        L.lomo_linear_forward(dev(X), dev(W), Y.t)
    x, w, r = X.astype(np.float64), W.astype(np.float64), R.astype(np.float64) if residual else 0.0
    product_ok(Y.host(), x @ w.T + r, np.abs(x) @ np.abs(w).T + np.abs(r), "Y")


# (T, K, N): tiles of the product, of the product with a residual
FORWARD_TILES = {(129, 520, 248): ((64, 64), (64, 64)), (264, 1032, 4104): ((128, 64), (128, 64)), (520, 2056, 2056): ((128, 64), (128, 64)),
                 (504, 1032, 5512): ((128, 128), (128, 128)), (1016, 2056, 3080): ((128, 128), (128, 128)),
                 (3080, 104, 4104): ((256, 256), (256, 256))}


@pytest.mark.parametrize("T,K,N", FORWARD_TILES)
@pytest.mark.parametrize("residual", ["none", "own buffer", "in place"])
def test_forward_in_each_tile_shape(L, T, K, N, residual):
    # the product with a residual has the form and the epilogue of an update of an N x T output over K indices
    forward, update = L.KERNEL_FAMILIES.index("forward"), L.KERNEL_FAMILIES.index("wgrad_update")
    got = L.lomo_contraction_tiles(forward, [(T, K, N)])[0], L.lomo_contraction_tiles(update, [(K, N, T)])[0]
    assert got == FORWARD_TILES[T, K, N], "this shape no longer exercises the kernels it is here for: choose another"
    X, W, R = f16(14, (T, K), 1.0), f16(15, (N, K), 0.05), f16(16, (T, N), 1.0)
    Y = Guarded((T, N), R if residual == "in place" else None)
    if residual == "none":
        L.lomo_linear_forward(dev(X), dev(W), Y.t)
    elif residual == "in place":
        L.lomo_linear_forward(dev(X), dev(W), Y.t, True)
    else:
        L.lomo_linear_forward_residual(dev(X), dev(W), dev(R), Y.t)
    x, w, r = X.astype(np.float64), W.astype(np.float64), 0.0 if residual == "none" else R.astype(np.float64)
    product_ok(Y.host(), x @ w.T + r, np.abs(x) @ np.abs(w).T + np.abs(r), "Y")


# 64 x 64 tiles, then 128 x 64, 128 x 128 and 256 x 256 in both products
@pytest.mark.parametrize("T,K,N", [(70, 264, 72), (300, 520, 1032), (33, 256, 40), (520, 2056, 2056), (1016, 2056, 3080),
                                   (3080, 3336, 3848)])
def test_non_finite_rows_stay_in_their_rows(L, T, K, N):
    """The contraction lengths are not whole slices, so a short slice ends where the next row begins: an infinite row
    must not reach its neighbours' sums (0 * inf), forwards or backwards."""
    dY, W, X = f16(7, (T, N), 1.0), f16(8, (N, K), 0.05), f16(9, (T, K), 1.0)
    for bad in (0, T // 2, T - 1):
        d, x = dY.copy(), X.copy()
        d[bad], x[bad] = np.inf, np.nan
        dX, Y = Guarded((T, K)), Guarded((T, N))
        L.lomo_linear_dgrad(dev(d), dev(W), dX.t)
        L.lomo_linear_forward(dev(x), dev(W), Y.t)
        others = np.arange(T) != bad
        w = W.astype(np.float64)
        got_dx, got_y = dX.host(), Y.host()
        assert not np.isfinite(got_dx[bad]).any() and not np.isfinite(got_y[bad]).any()
        a, b = dY[others].astype(np.float64), X[others].astype(np.float64)
        product_ok(got_dx[others], a @ w, np.abs(a) @ np.abs(w), "dX")
        product_ok(got_y[others], b @ w.T, np.abs(b) @ np.abs(w).T, "Y")


def test_bits_do_not_depend_on_the_size_of_the_call(L):
    """Every element is one chain of fp32 sums over the contraction, in the same order in every kernel: a token's Y and dX
    have the same bits in a batch of 3080 as in one of 8, a row of W the same update in a tensor of 4104 rows as in one of
    8.  The sizes take the call through all tile shapes; none of the contractions is a whole number of slices."""
    T, K, N = 3080, 1032, 4104
    X, dY, W, R = dev(f16(10, (T, K), 1.0)), dev(f16(11, (T, N), 1.0)), dev(f16(12, (N, K), 0.02)), dev(f16(13, (T, N), 1.0))
    new = lambda *shape: torch.empty(*shape, dtype=torch.float16, device=DEV)

    def by_token(rows):
        x, d, r = X[rows].contiguous(), dY[rows].contiguous(), R[rows].contiguous()
        n = x.shape[0]
        Y, Y2, dX = new(n, N), new(n, N), new(n, K)
        L.lomo_linear_forward(x, W, Y)
        L.lomo_linear_forward_residual(x, W, r, Y2)
        L.lomo_linear_dgrad(d, W, dX)
        return Y, Y2, dX

    def by_feature(rows):
        d, w, w2 = dY[:, rows].contiguous(), W[rows].clone(), W[rows].clone()
        flag = torch.zeros(1, dtype=torch.int32, device=DEV)
        L.lomo_linear_backward_update(X, d, w, None, 1e-4, 1.0, 1.0)
        L.lomo_linear_backward_update_clip_value(X, d, w2, None, 1e-4, 1.0, 30.0, flag)
        return w, w2

    tiles = {part: {L.lomo_contraction_tiles(L.KERNEL_FAMILIES.index(f), [shape(n)])[0] for n in (8, 72, 264, 776, 1544, whole)}
             for part, f, shape, whole in (("Y", "forward", lambda n: (n, K, N), T), ("dX", "dgrad", lambda n: (n, K, N), T),
                                           ("W", "wgrad_update", lambda n: (T, K, n), N))}
    assert tiles["Y"] == {(64, 64), (128, 64), (128, 128), (256, 256)} and len(tiles["dX"]) > 1 and len(tiles["W"]) > 2, tiles
    for part, total, size in ((by_token, T, 1), (by_feature, N, 8)):
        whole = part(slice(0, total))
        for count in (size, 8, 72, 264, 776, 1544):
            rows = slice(total - count, total)
            for k, (a, b) in enumerate(zip(part(rows), whole)):
                assert torch.equal(a.view(torch.int16), b[rows].view(torch.int16)), (part.__name__, count, k)


# X, dY or W between 2 GiB and the 3.5 GiB that a descriptor covers, and beyond; the last contraction index is not the end of
# a slice.  (T, K, N)
@pytest.mark.parametrize("T,K,N", [(41003, 264, 32000), (60003, 264, 32000), (60003, 32008, 264)])
def test_large_activations(L, T, K, N):
    """Update and norm: bit for bit those of pieces of the output, whose operands are small, and sampled against 64 bits."""
    gen = torch.Generator(device=DEV).manual_seed(T + K)
    X = torch.randn(T, K, generator=gen, device=DEV, dtype=torch.float16)
    dY = torch.randn(T, N, generator=gen, device=DEV, dtype=torch.float16)
    W, s = torch.zeros(N, K, device=DEV, dtype=torch.float16), 2.0 ** -5
    acc, flag = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    L.lomo_wgrad_sqnorm(X, dY, acc, flag)
    L.lomo_linear_backward_update(X, dY, W, None, s, 1.0, 1.0, flag)
    assert int(flag.item()) == 0
    by_rows, step = N > K, 4000
    total = 0.0
    for at in range(0, max(N, K), step):
        cut = slice(at, at + step)
        x, d, w = (X, dY[:, cut].contiguous(), W[cut]) if by_rows else (X[:, cut].contiguous(), dY, W[:, cut])
        W2, acc2 = torch.zeros(w.shape, device=DEV, dtype=torch.float16), torch.zeros(1, dtype=torch.float64, device=DEV)
        L.lomo_linear_backward_update(x, d, W2, None, s, 1.0, 1.0)
        L.lomo_wgrad_sqnorm(x, d, acc2)
        total += float(acc2.item())
        assert torch.equal(W2.view(torch.int16), w.contiguous().view(torch.int16)), at
    assert abs(float(acc.item()) / total - 1) < 1e-6
    n, k = [0, 17, N // 2, N - 1], [0, 9, K // 2, K - 1]
    d, x = dY[:, n].double().cpu().numpy(), X[:, k].double().cpu().numpy()
    product_ok(W[n][:, k].cpu().numpy(), -s * (d.T @ x), s * (np.abs(d).T @ np.abs(x)), "W")
    dY[T - 1, N - 1] = np.inf                  # the very last element is still read
    L.lomo_wgrad_sqnorm(X, dY, acc, flag)
    assert int(flag.item()) == 1


@pytest.mark.parametrize("T,K,N", [(264, 16384, 70008), (264, 16384, 128264)])
def test_large_weights(L, T, K, N):
    gen = torch.Generator(device=DEV).manual_seed(N)
    dY = torch.randn(T, N, generator=gen, device=DEV, dtype=torch.float16)
    W = torch.randn(N, K, generator=gen, device=DEV, dtype=torch.float16).mul_(0.02)
    dX = torch.empty(T, K, device=DEV, dtype=torch.float16)
    L.lomo_linear_dgrad(dY, W, dX)
    for at in range(0, K, 4096):
        piece = torch.empty(T, 4096, device=DEV, dtype=torch.float16)
        L.lomo_linear_dgrad(dY, W[:, at:at + 4096].contiguous(), piece)
        assert torch.equal(piece.view(torch.int16), dX[:, at:at + 4096].contiguous().view(torch.int16)), at
    t, k = [0, 100, T - 1], [0, 9, K // 2, K - 1]
    d, w = dY[t].double().cpu().numpy(), W[:, k].double().cpu().numpy()
    product_ok(dX[t][:, k].cpu().numpy(), d @ w, np.abs(d) @ np.abs(w), "dX")
