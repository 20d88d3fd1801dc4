"""The autotuner keeps the defaults unless a candidate beats them by a margin."""
import pytest

from paper_1109_3739_amd import autotune

INF = float("inf")


@pytest.mark.parametrize("results,chosen", [
    ([(1.0, {}), (0.99, {"tiny_max": 32})], {}),
    ([(1.0, {}), (0.97, {"tiny_max": 32})], {"tiny_max": 32}),
    ([(1.0, {}), (0.97, {"tiny_max": 32}), (0.9, {"count_threads": 512})], {"count_threads": 512}),
    ([(1.0, {}), (INF, {"tiny_max": 32, "error": "x"})], {}),
    ([(INF, {}), (0.5, {"tiny_max": 32})], {"tiny_max": 32}),  # defaults that fail
    ([(1.0, {"tiny_max": 32}), (0.99, {"count_threads": 512})], {"count_threads": 512}),  # no defaults among them
])
def test_pick(results, chosen):
    assert autotune.pick(results)[1] == chosen


def test_candidates_differ_in_effect():
    # up to 512 products single_part_max makes no difference, so smaller values would be tried twice
    assert all(c.get("single_part_max", 1024) >= 512 for c in autotune.CANDIDATES)
    assert len({tuple(sorted(c.items())) for c in autotune.CANDIDATES}) == len(autotune.CANDIDATES)
