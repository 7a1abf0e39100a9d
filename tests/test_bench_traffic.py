"""The bench line's HBM traffic is per launch as its other figures are: from a counter summary of a pass with as many launches."""
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_traffic_is_of_the_launches_that_are_timed():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    for workload, launches, algorithmic in (("llama7b_stack", 8, 45006 * 2 ** 20), ("llama7b_layer", 2, 1382 * 2 ** 20)):
        traffic, source = bench.profiled_traffic(workload, launches)
        assert os.path.exists(os.path.join(ROOT, source))
        assert 2.0 < traffic * launches / algorithmic < 3.0
        assert bench.profiled_traffic(workload, launches - 1) == (None, None)
    assert bench.profiled_traffic("linear1024", 1) == (None, None)
