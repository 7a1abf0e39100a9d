"""Which shape of tile the contractions of a call take (host function, no GPU): alone, a tensor of few tiles takes small ones; in
a list whose tensors fill the chip together, all stay in the persistent kernel, except a long contraction of few tiles."""
import time

import pytest

import paper_2306_09782_amd as L

UPDATE, NORM, DGRAD, FORWARD = (L.KERNEL_FAMILIES.index(k) for k in ("wgrad_update", "wgrad_sqnorm", "dgrad", "forward"))


def layer_stack(H, F, T, layers):
    return ([(T, F, H), (T, H, F), (T, H, F)] + [(T, H, H)] * 4) * layers


@pytest.mark.parametrize("H,F,T,layers", [(4096, 11008, 1024, 4), (4096, 11008, 2048, 2), (4096, 11008, 1024, 32),
                                          (5120, 13824, 1024, 3), (5120, 13824, 4096, 3), (8192, 22016, 2048, 1),
                                          (2048, 5504, 2048, 8), (2048, 5504, 1000, 8), (1024, 2816, 512, 24),
                                          (1024, 2816, 2048, 24), (1024, 2816, 4096, 24)])
@pytest.mark.parametrize("family", [UPDATE, NORM, DGRAD])
def test_lists_that_fill_the_chip_stay_together(H, F, T, layers, family):
    assert set(L.lomo_contraction_tiles(family, layer_stack(H, F, T, layers))) == {(256, 256)}


@pytest.mark.parametrize("family,H,F,T,layers,vocabulary", [(DGRAD, 5120, 13824, 2100, 1, 0), (DGRAD, 5120, 13824, 1070, 3, 32000),
                                                            (UPDATE, 1024, 2816, 6000, 2, 32000), (NORM, 1024, 2816, 6000, 2, 32000)])
def test_a_gain_within_the_error_of_the_times_splits_no_list(family, H, F, T, layers, vocabulary):
    shapes = layer_stack(H, F, T, layers) + [(T, H, vocabulary)] * bool(vocabulary)
    assert set(L.lomo_contraction_tiles(family, shapes)) == {(256, 256)}


@pytest.mark.parametrize("family,shape", [(UPDATE, (512, 1024, 1024)), (NORM, (512, 1024, 1024)), (DGRAD, (512, 1024, 1024)),
                                          (FORWARD, (256, 1024, 3072)), (DGRAD, (1024, 4096, 4096)), (DGRAD, (256, 1024, 32000))])
def test_a_tensor_of_few_tiles_takes_small_ones_alone(family, shape):
    assert L.lomo_contraction_tiles(family, [shape])[0] != (256, 256)


@pytest.mark.parametrize("family,shape", [(UPDATE, (4096, 4096, 11008)), (NORM, (4096, 4096, 4096)), (DGRAD, (4096, 11008, 4096)),
                                          (FORWARD, (8192, 4096, 12288)), (UPDATE, (1024, 4096, 32000))])
def test_a_tensor_of_many_tiles_takes_large_ones_alone(family, shape):
    assert L.lomo_contraction_tiles(family, [shape]) == [(256, 256)]


def test_only_the_long_contraction_leaves_a_list():
    stack = layer_stack(1024, 2816, 512, 24)
    *rest, vocabulary = L.lomo_contraction_tiles(DGRAD, stack + [(512, 1024, 32000)])
    assert set(rest) == {(256, 256)} and vocabulary != (256, 256)


@pytest.mark.parametrize("family,shape", [(UPDATE, (65536, 4096, 32000)), (NORM, (60000, 264, 32000)), (UPDATE, (60000, 32008, 264)),
                                          (DGRAD, (264, 16384, 128256)), (FORWARD, (65536, 32000, 8))])
def test_operands_larger_than_a_descriptor_covers(family, shape):
    """More than 3.5 GiB of X, dY or W: the persistent kernel, whose descriptors move with the walk."""
    assert L.lomo_contraction_tiles(family, [shape])[0] == ((256, 256) if family != FORWARD else (64, 64))


def test_only_very_long_rows_leave_the_kernels_with_descriptors():
    for family in (UPDATE, NORM, DGRAD, FORWARD):
        assert L.lomo_contraction_tiles(family, [(8, 9_000_000, 8)]) == [(0, 0)]
        assert L.lomo_contraction_tiles(family, [(8, 7_000_000, 8)])[0] != (0, 0)


def test_host_time_of_a_list_of_many_shapes():
    """The choice for a list of 60 different shapes takes about as long as 60 choices for one of them; reckoning the whole pass
    again for every move that is tried took five times as long, half that before there were six shapes of tile."""
    shapes = [(1024, 8 * (100 + 37 * i % 1400), 8 * (100 + 91 * i % 1400)) for i in range(60)]

    def least(f):
        times = []
        for _ in range(20):
            begin = time.perf_counter()
            f()
            times.append(time.perf_counter() - begin)
        return min(times)

    assert least(lambda: L.lomo_contraction_tiles(DGRAD, shapes)) < 2.5 * least(lambda: [L.lomo_contraction_tiles(DGRAD, [s]) for s in shapes])


def test_bad_arguments():
    assert L.lomo_contraction_tiles(UPDATE, []) == []
    for family, shape in ((UPDATE, (0, 8, 8)), (L.KERNEL_FAMILIES.index("embedding"), (8, 8, 8))):
        with pytest.raises(L.LomoError):
            L.lomo_contraction_tiles(family, [shape])
