"""256 x 128 tiles, ragged on both sides and in the contraction: all products against the oracle, with the bars of
test_gpu_edges.py, and rows of the result against the bits that they have in a call of eight rows."""
import numpy as np
import pytest
import torch

from test_gpu_edges import DEV, Guarded, L, dev, f16, product_ok, step_matches_oracle  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,N", [(2040, 2056, 2056), (1000, 1032, 5128), (1544, 4104, 1032)])
def test_step(L, T, K, N):
    tiles = {f: L.lomo_contraction_tiles(L.KERNEL_FAMILIES.index(f), [(T, K, N)])[0] for f in ("dgrad", "wgrad_update", "wgrad_sqnorm")}
    assert tiles["wgrad_update"] == tiles["wgrad_sqnorm"] == (256, 128) and (T != 2040 or tiles["dgrad"] == (256, 128))
    step_matches_oracle(L, T, K, N)


@pytest.mark.parametrize("T,K,N", [(1000, 2056, 5128), (2040, 2056, 2056)])
@pytest.mark.parametrize("residual", [False, True])
def test_forward(L, T, K, N, residual):
    assert L.lomo_contraction_plan(L.KERNEL_FAMILIES.index("forward"), [(T, K, N)], residual)[0] == [(256, 128)]
    X, W, R = f16(31, (T, K), 1.0), f16(32, (N, K), 0.05), f16(33, (T, N), 1.0)
    Y, few = Guarded((T, N)), torch.empty(8, N, dtype=torch.float16, device=DEV)
    if residual:
        L.lomo_linear_forward_residual(dev(X), dev(W), dev(R), Y.t)
        L.lomo_linear_forward_residual(dev(X[-8:]), dev(W), dev(R[-8:]), few)
    else:
        L.lomo_linear_forward(dev(X), dev(W), Y.t)
        L.lomo_linear_forward(dev(X[-8:]), dev(W), few)
    assert torch.equal(Y.t[-8:].view(torch.int16), few.view(torch.int16))
    x, w, r = X.astype(np.float64), W.astype(np.float64), R.astype(np.float64) if residual else 0.0
    product_ok(Y.host(), x @ w.T + r, np.abs(x) @ np.abs(w).T + np.abs(r), "Y")
