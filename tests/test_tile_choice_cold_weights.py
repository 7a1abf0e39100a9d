"""Which shape of tile stored products take when their weights come from HBM (host function, no GPU)."""
import pytest

import paper_2306_09782_amd as L

DGRAD = L.KERNEL_FAMILIES.index("dgrad")


# (T, K, N) of dX: the tile that measured fastest with weights that no cache holds
@pytest.mark.parametrize("shape,tile", [((512, 13824, 5120), (256, 128)), ((1024, 8192, 22016), (256, 128)), ((350, 13824, 5120), (256, 128)),
                                        ((234, 2048, 32000), (64, 32)), ((350, 4096, 32000), (128, 64)), ((700, 4096, 11008), (128, 128))])
def test_a_product_alone(shape, tile):
    assert L.lomo_contraction_tiles(DGRAD, [shape]) == [tile]


def test_long_contractions_of_a_list_share_one_launch():
    """Alone, the vocabulary takes 128 x 64 tiles; together with the layers its walk runs behind theirs."""
    T, H, F = 350, 4096, 11008
    stack = ([(T, F, H), (T, H, F), (T, H, F)] + [(T, H, H)] * 4) * 2 + [(T, H, 32000)]
    tiles = L.lomo_contraction_tiles(DGRAD, stack)
    assert {t for s, t in zip(stack, tiles) if s[2] > 4096 or s[1] > 4096} == {(128, 128)}
    assert L.lomo_contraction_tiles(DGRAD, [stack[-1]]) == [(128, 64)]
