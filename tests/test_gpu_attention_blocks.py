"""The attention kernels at the edges of their blocks and on both sides of the rule that splits a call: 128 rows per workgroup or 64 with
the tiles split over the waves, sequences that end in the middle of a block, one block alone.  Against 64 bits on the GPU, every
sequence and head by itself: fp16 outputs and fp16 P and dS are each off by at most half a unit in the last place, 2^-11 of
their size, so a head's relative error in the Frobenius norm stays below 2^-10.  (Element-wise bars: test_gpu_attention.py,
test_gpu_forward.py.)"""
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


def reference(q, k, v, do):
    """One head of one sequence in 64 bits: o, lse, dq, dk, dv."""
    s = q.shape[0]
    scores = (q @ k.t().contiguous()) / 128 ** 0.5
    scores = scores.masked_fill(torch.ones(s, s, device=DEV, dtype=torch.bool).triu(1), -float("inf"))
    P, lse = scores.softmax(-1), scores.logsumexp(-1)
    o = P @ v
    dS = P * (do @ v.t().contiguous() - (do * o).sum(-1, keepdim=True)) / 128 ** 0.5
    return o, lse, dS @ k, dS.t().contiguous() @ q, P.t().contiguous() @ do


# waves of 32 rows per call: 2 ... 34 (split), 1280 (forward not, backward split), 2048 and more (not split)
@pytest.mark.parametrize("B,s,nh", [(1, 64, 1), (2, 192, 1), (1, 1088, 1), (4, 320, 32), (32, 64, 32), (12, 192, 32), (8, 320, 32), (2, 1088, 32)])
def test_blocks(L, B, s, nh):
    T, H = B * s, nh * 128
    gen = torch.Generator(device=DEV).manual_seed(s + nh)
    normal = lambda *shape: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float16)
    qkv, do = normal(T, 3 * H), normal(T, H)
    guard = torch.full((T + 256, 3 * H), 9.0, dtype=torch.float16, device=DEV)      # rows in front of and behind the gradient
    o, grad = torch.full((T, H), 9.0, dtype=torch.float16, device=DEV), guard[128:128 + T]
    lse, delta = torch.empty(T, nh, device=DEV), torch.empty(T, nh, device=DEV)
    L.lomo_attention_forward(qkv, o, lse, B, s, nh)
    L.lomo_attention_backward(qkv, o, do, lse.view(-1), None, None, delta.view(-1), grad, B, s, nh)
    assert bool((guard[:128] == 9).all()) and bool((guard[128 + T:] == 9).all())
    off = lambda got, want: float((got.double() - want).norm() / want.norm())
    for b in sorted({0, B // 2, B - 1}):
        for n in sorted({0, nh // 2, nh - 1}):
            rows, cols = slice(b * s, (b + 1) * s), slice(n * 128, (n + 1) * 128)
            part = lambda x, i: x[rows, i * H + n * 128:i * H + (n + 1) * 128].double()
            want = reference(part(qkv, 0), part(qkv, 1), part(qkv, 2), do[rows, cols].double())
            assert float((lse[rows, n].double() - want[1]).abs().max()) < 1e-5
            got = (o[rows, cols], None, *(grad[rows, i * H + n * 128:i * H + (n + 1) * 128] for i in range(3)))
            for name, g, w in zip(("o", "lse", "dq", "dk", "dv"), got, want):
                if g is not None:
                    assert off(g, w) < 2.0 ** -10, (name, b, n, off(g, w))


@pytest.mark.parametrize("B,nh,rope", [(1, 1, True), (3, 7, True), (8, 4, False), (130, 32, True)])
def test_sequence_of_one_block_against_longer_ones(L, B, nh, rope):
    """Sequences of one block have a backward kernel of their own.  In sequences of two, dq of the first block depends on that block alone
    and dk, dv of the second on the second alone (given o and lse), so the kernels for longer sequences give the same bits there."""
    s, H = 64, nh * 128
    gen = torch.Generator(device=DEV).manual_seed(B + nh)
    normal = lambda *shape: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float16)
    qkv, do = normal(B, 2 * s, 3 * H), normal(B, 2 * s, H)
    angle = torch.rand(2 * s, 64, generator=gen, device=DEV)
    table = (angle.cos(), angle.sin()) if rope else (None, None)

    def backward(rows):
        part = lambda x: x[:, rows].contiguous()
        n = part(qkv).shape[1]
        guard = torch.full((B * n + 256, 3 * H), 9.0, dtype=torch.float16, device=DEV)      # rows in front of and behind the gradient
        delta, grad = torch.full((B * n, nh), 9.0, device=DEV), guard[128:128 + B * n]
        L.lomo_attention_backward(part(qkv).view(B * n, -1), part(o).view(B * n, -1), part(do).view(B * n, -1), part(lse).view(-1),
                                  *(None if x is None else x[rows].contiguous() for x in table), delta.view(-1), grad, B, n, nh)
        assert bool((guard[:128] == 9).all()) and bool((guard[128 + B * n:] == 9).all())
        return delta.view(B, n, nh), grad.view(B, n, 3, H)

    o, lse = torch.empty(B, 2 * s, H, dtype=torch.float16, device=DEV), torch.empty(B, 2 * s, nh, device=DEV)
    L.lomo_attention_forward(qkv.view(2 * B * s, -1), o.view(2 * B * s, -1), lse.view(2 * B * s, -1), B, 2 * s, nh)
    delta, grad = backward(slice(0, 2 * s))
    for rows, of_block in ((slice(0, s), slice(0, 1)), (slice(s, 2 * s), slice(1, 3))):
        one_delta, one = backward(rows)
        assert torch.equal(one_delta, delta[:, rows])
        assert torch.equal(one[:, :, of_block].view(torch.int16), grad[:, rows, of_block].view(torch.int16))


def test_rows_beyond_32_bit_offsets(L):
    """More heads than a wave's 32-bit offsets reach over four rows (48 GiB of q, k and v, most of it never looked at)."""
    s, nh = 64, (1 << 20) + 8
    qkv = torch.empty(s, 3, nh, 128, dtype=torch.float16, device=DEV)
    o, lse = torch.empty(s, nh, 128, dtype=torch.float16, device=DEV), torch.empty(s, nh, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(3)
    heads = (0, 1, nh // 2 + 5, nh - 1)
    for n in heads:
        qkv[:, :, n] = torch.randn(s, 3, 128, generator=gen, device=DEV, dtype=torch.float16)
    L.lomo_attention_forward(qkv.view(s, -1), o.view(s, -1), lse, 1, s, nh)
    for n in heads:
        q, k, v = (qkv[:, i, n].contiguous() for i in range(3))
        one, one_lse = torch.empty(s, 128, dtype=torch.float16, device=DEV), torch.empty(s, 1, device=DEV)
        L.lomo_attention_forward(torch.cat((q, k, v), 1), one, one_lse, 1, s, 1)
        assert torch.equal(one, o[:, n]) and torch.equal(one_lse[:, 0], lse[:, n]), n
        want = reference(q.double(), k.double(), v.double(), q.double())[0]
        assert float((one.double() - want).norm() / want.norm()) < 2.0 ** -10
    del qkv, o, lse
    torch.cuda.empty_cache()
