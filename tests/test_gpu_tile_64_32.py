"""64 x 32 tiles, which long contractions of few tiles take: ragged on both sides and in the contraction, against 64 bits with the
bars of test_gpu_edges.py, and against the bits of the same rows in a call of larger tiles."""
import numpy as np
import pytest
import torch

from test_gpu_edges import DEV, Guarded, L, dev, f16, product_ok  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,M,C", [(200, 520, 5128), (8, 520, 4616), (33, 1000, 4680), (256, 1024, 8192)])
@pytest.mark.parametrize("product", ["dgrad", "forward"])
def test_product(L, T, M, C, product):
    shape = lambda t: (t, M, C) if product == "dgrad" else (t, C, M)
    family = L.KERNEL_FAMILIES.index(product)
    assert L.lomo_contraction_tiles(family, [shape(T)]) == [(64, 32)] and L.lomo_contraction_tiles(family, [shape(2000)]) != [(64, 32)]
    B, W = f16(51, (2000, C), 1.0), f16(52, (C, M) if product == "dgrad" else (M, C), 0.05)
    call = L.lomo_linear_dgrad if product == "dgrad" else L.lomo_linear_forward
    few, many = Guarded((T, M)), torch.empty(2000, M, dtype=torch.float16, device=DEV)
    call(dev(B[:T]), dev(W), few.t)
    call(dev(B), dev(W), many)
    assert torch.equal(few.t.view(torch.int16), many[:T].view(torch.int16))
    b, w = B[:T].astype(np.float64), W.astype(np.float64) if product == "dgrad" else W.astype(np.float64).T
    product_ok(few.host(), b @ w, np.abs(b) @ np.abs(w), product)


def test_non_finite_rows_stay_in_their_rows(L):
    T, M, C = 70, 264, 5000
    assert L.lomo_contraction_tiles(L.KERNEL_FAMILIES.index("dgrad"), [(T, M, C)]) == [(64, 32)]
    B, W = f16(53, (T, C), 1.0), f16(54, (C, M), 0.05)
    for bad in (0, T // 2, T - 1):
        b = B.copy()
        b[bad] = np.inf
        out = Guarded((T, M))
        L.lomo_linear_dgrad(dev(b), dev(W), out.t)
        others = np.arange(T) != bad
        got, x, w = out.host(), B[others].astype(np.float64), W.astype(np.float64)
        assert not np.isfinite(got[bad]).any()
        product_ok(got[others], x @ w, np.abs(x) @ np.abs(w), "dX")
