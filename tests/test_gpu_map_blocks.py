"""Contraction maps around the 64-vertex blocks that rows are mapped through
and the aggregates that columns are taken from without counting."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu


def _maps(n):
    v = np.arange(n)
    return {
        "runs": v // 5,
        "one": v * 0,
        "each": v,
        "skip_in_block": v // 5 + 3 * (v >= min(100, n // 2)),
        "skip_between_blocks": v // 7 + 2 * (v >= 64),
        "first_empty": v // 3 + 4,
        "drop_at_block": np.where(v < 64, v // 4 + 1, v // 8),
    }


@pytest.mark.parametrize("n", [1, 64, 65, 130, 1000])
@pytest.mark.parametrize("name", sorted(_maps(1)))
def test_maps(spx, n, name):
    import torch
    agg = _maps(n)[name]
    A = W.erdos_renyi(n, n, min(6, n), seed=n, values="f64")
    A.num = np.random.default_rng(n).integers(1, 9, A.ir.size).astype(np.int64)
    dA, dagg = spx.from_host(A), torch.from_numpy(agg.astype(np.int32)).cuda()
    for nc in (int(agg.max()) + 1, int(agg.max()) + 8):  # the last aggregates empty, too
        got = spx.contract(dA, dagg, nc, dagg, nc).to_host_csc()
        assert_same_csc(got, oracle.contract(A, agg, nc, agg, nc, "plus_times"), exact_values=True, what=f"{name} {n} {nc}")
