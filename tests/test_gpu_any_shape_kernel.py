"""The register-staged contraction kernel, which serves rows too long for the direct-to-LDS kernels' 32-bit offsets.  It adds in
the same order as they do, so its results are held to theirs bit for bit: at ordinary shapes by a child process in whose
environment LOMO_DISABLE_FAST=1 takes every contraction to it, and at rows of nine million elements, which nothing else
serves, against pieces of the output that the others compute."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HERE = os.path.dirname(os.path.abspath(__file__))

# (T, K, N): the smallest, edges of its 128 x 128 and 256 x 256 tiles and of its slices, whole tiles; from 192 tiles of
# 256 x 256 on it takes those: (300, 3080, 4104) in the update, (3336, 3848, 264) in dX, (3336, 264, 3848) in Y
SHAPES = [(1, 8, 8), (33, 248, 520), (64, 128, 256), (129, 136, 120), (257, 72, 1032), (777, 1544, 1032), (300, 3080, 4104),
          (3336, 3848, 264), (3336, 264, 3848)]


@pytest.fixture(scope="module")
def L():
    import paper_2306_09782_amd as L
    if not os.path.exists(L.library_path()):
        from paper_2306_09782_amd.build import build
        build(verbose=False)
    L.load_library()
    return L


def all_products(L, T, K, N):
    gen = torch.Generator().manual_seed(T * 3 + K * 5 + N)
    normal = lambda shape, sigma: (torch.randn(shape, generator=gen) * sigma).half().to(DEV)
    X, dY, W, R = normal((T, K), 1.0), normal((T, N), 1.0), normal((N, K), 0.02), normal((T, N), 1.0)
    new = lambda *shape: torch.full(shape, 7.0, dtype=torch.float16, device=DEV)
    acc, flags = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(2, dtype=torch.int32, device=DEV)
    Y, Y2, Y3, dX, W2, W3 = new(T, N), new(T, N), R.clone(), new(T, K), W.clone(), W.clone()
    L.lomo_linear_forward(X, W, Y)
    L.lomo_linear_forward_residual(X, W, R, Y2)
    L.lomo_linear_forward(X, W, Y3, True)
    L.lomo_linear_dgrad(dY, W, dX)
    L.lomo_wgrad_sqnorm(X, dY, acc, flags[:1])
    L.lomo_linear_backward_update(X, dY, W2, None, 1e-3, 1.0, 1.0)
    L.lomo_linear_backward_update_clip_value(X, dY, W3, None, 1e-3, 1.0, float(T) ** 0.5, flags[1:])
    out = {"Y": Y, "Y + R": Y2, "Y onto R": Y3, "dX": dX, "W": W2, "W by value": W3}
    out = {k: v.cpu().numpy().view(np.uint16) for k, v in out.items()}
    return {**out, "sqnorm": acc.cpu().numpy(), "flags": flags.cpu().numpy()}


def child(path):
    import paper_2306_09782_amd as L
    np.savez(path, **{f"{i} {k}": v for i, s in enumerate(SHAPES) for k, v in all_products(L, *s).items()})


def test_it_gives_the_bits_of_the_other_kernels(L, tmp_path):
    path = str(tmp_path / "products.npz")
    env = dict(os.environ, LOMO_DISABLE_FAST="1", PYTHONPATH=os.pathsep.join([os.path.dirname(HERE), HERE]))
    code = f"import test_gpu_any_shape_kernel as t; t.child({path!r})"
    res = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stderr[-2000:]
    got = np.load(path)
    for i, shape in enumerate(SHAPES):
        for k, want in all_products(L, *shape).items():
            if k == "sqnorm":                  # its tiles differ, and a tile's sum of squares is an fp32 sum
                assert abs(float(got[f"{i} {k}"][0]) / float(want[0]) - 1) < 1e-6, shape
            else:
                np.testing.assert_array_equal(got[f"{i} {k}"], want, err_msg=f"{k} {shape}")


def test_rows_of_nine_million_elements(L):
    T, K, N = 8, 9_000_000, 24
    update, norm, dgrad, forward = (L.KERNEL_FAMILIES.index(k) for k in ("wgrad_update", "wgrad_sqnorm", "dgrad", "forward"))
    for family in (update, norm, dgrad, forward):
        assert L.lomo_contraction_tiles(family, [(T, K, N)]) == [(0, 0)]
    gen = torch.Generator(device=DEV).manual_seed(3)
    normal = lambda *shape: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float16)
    X, dY, W = normal(T, K), normal(T, N), normal(N, K)
    dX, Y, W2 = torch.empty_like(X), torch.empty_like(dY), W.clone()
    acc, acc2 = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(1, dtype=torch.float64, device=DEV)
    L.lomo_linear_dgrad(dY, W, dX)
    L.lomo_linear_forward(X, W, Y)
    L.lomo_wgrad_sqnorm(X, dY, acc)
    L.lomo_linear_backward_update(X, dY, W2, None, 1e-2, 1.0, 1.0)
    for at in range(0, K, K // 3):
        cut = slice(at, at + K // 3)
        x, w = X[:, cut].contiguous(), W[:, cut].contiguous()
        piece = torch.empty_like(x)
        assert L.lomo_contraction_tiles(dgrad, [(T, x.shape[1], N)]) != [(0, 0)]
        L.lomo_linear_dgrad(dY, w, piece)
        L.lomo_wgrad_sqnorm(x, dY, acc2)
        L.lomo_linear_backward_update(x, dY, w, None, 1e-2, 1.0, 1.0)
        assert torch.equal(piece.view(torch.int16), dX[:, cut].contiguous().view(torch.int16)), at
        assert torch.equal(w.view(torch.int16), W2[:, cut].contiguous().view(torch.int16)), at
    assert abs(float(acc.item()) / float(acc2.item()) - 1) < 1e-6
    # Y: 562 500 additions one behind the other, each off by up to a unit of the partial sum's last place (2^-23 of about 5000):
    # 0.45 if they err at random (562 500^0.5 units), 335 if all one way.  The bar is that of the suite's other cancelling sums,
    # 2^-20 of the sum of the absolute products (here 5.5), and half an fp16 step for the rounding of the result.
    x, w = X.double(), W.double()
    want = torch.stack([(x * w[n]).sum(1) for n in range(N)], 1)
    mag = torch.stack([(x * w[n]).abs().sum(1) for n in range(N)], 1)
    off = (Y.double() - want).abs() - 2.0 ** -11 * want.abs()
    assert bool((off <= 2.0 ** -20 * mag).all()), float((off / mag).max())
