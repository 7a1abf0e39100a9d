"""The persistent kernel of products with a contraction-contiguous operand walks the contraction in slots of 64 indices, two per
trip: lengths one step off a slot, an even and an odd number of slots, and less than one, in tiles that are cut off on both
sides.  Every element is one chain of sums in the order of the other kernels, so the last rows are held to the bits that they have
in a call of eight rows (64 x 64 tiles), and sampled rows to 64 bits with the bar of test_gpu_edges.py."""
import os

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def L():
    import paper_2306_09782_amd as L
    if not os.path.exists(L.library_path()):
        from paper_2306_09782_amd.build import build
        build(verbose=False)
    L.load_library()
    return L


@pytest.mark.parametrize("C", [8, 56, 64, 72, 120, 128, 136, 192, 200, 256])
@pytest.mark.parametrize("product", ["forward", "residual", "dgrad"])
def test_slots(L, product, C):
    T, M = 3080, 4104                                  # rows of the output, columns of the output
    K, N = (M, C) if product == "dgrad" else (C, M)
    family = L.KERNEL_FAMILIES.index("dgrad" if product == "dgrad" else "forward")
    if C > 8:                                          # one short chain may go to small tiles
        assert L.lomo_contraction_plan(family, [(T, K, N)], product == "residual")[0] == [(256, 256)]
    gen = torch.Generator(device=DEV).manual_seed(C)
    normal = lambda *shape: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float16)
    B, W, R = normal(T, C), normal(N, K), normal(T, M)

    def run(rows):
        b, out = B[rows].contiguous(), torch.full((len(range(*rows.indices(T))), M), 7.0, dtype=torch.float16, device=DEV)
        if product == "dgrad":
            L.lomo_linear_dgrad(b, W, out)
        elif product == "forward":
            L.lomo_linear_forward(b, W, out)
        else:
            L.lomo_linear_forward_residual(b, W, R[rows].contiguous(), out)
        return out

    whole, few = run(slice(0, T)), run(slice(T - 8, T))
    assert torch.equal(whole[-8:].view(torch.int16), few.view(torch.int16))
    pick = torch.tensor([0, 255, 256, 1700, T - 1], device=DEV)
    b, w = B[pick].double(), W.double() if product == "dgrad" else W.double().t().contiguous()
    want, mag = b @ w, b.abs() @ w.abs()
    if product == "residual":
        want, mag = want + R[pick].double(), mag + R[pick].double().abs()
    off = (whole[pick].double() - want).abs()
    assert bool((off <= 2.0 ** -11 * want.abs() + 2.0 ** -20 * mag).all())
