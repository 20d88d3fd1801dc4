"""Columns of at most 64 products: groups of 16, 32 and 64 lanes, B entries in
blocks of every width, and columns whose products are listed instead."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu

# lengths of the A columns that one column of C takes
PICKS = [[1], [16], [17], [32], [33], [64], [63, 1], [1, 63], [2] * 8, [1] * 16, [1] * 17, [1] * 32, [1] * 33, [1] * 64,
         [4, 4, 4, 4], [4, 4, 4, 5], [4, 5, 4, 4], [8] * 8, [7] * 8, [8] * 7 + [7], [6] * 7 + [9], [0] * 20 + [3],
         [0] * 70 + [2, 5], [15, 1], [9, 7], [16, 16], [31, 1], [3, 0, 5, 0, 7], [32, 32], [20, 20, 20]]


@pytest.mark.parametrize("m", [70, (1 << 25) + 9])  # many equal rows; rows too long for 32-bit sort keys
@pytest.mark.parametrize("semiring,values", [("plus_times", "f64"), ("plus_times", "i64"), ("min_plus", "f32"),
                                             ("or_and", "none")])
def test_tiny_columns(spx, m, semiring, values):
    rng = np.random.default_rng(m + len(values))

    def num(n):
        return rng.integers(1, 100, n) if values == "i64" else rng.random(n).astype("f4" if values == "f32" else "f8")

    picks = [p for _ in range(9) for p in (PICKS[i] for i in rng.permutation(len(PICKS)))]
    lens = [d for p in picks for d in p]
    near = np.sort(rng.choice(m, 70, replace=False))  # equal rows also where there are many rows
    rows = [np.sort(rng.choice(near, d, replace=False)) for d in lens]
    A = W.from_triples(np.concatenate(rows), np.repeat(np.arange(len(lens)), lens), num(sum(lens)), m, len(lens))
    B = W.from_triples(np.arange(len(lens)), np.repeat(np.arange(len(picks)), [len(p) for p in picks]), num(len(lens)),
                       len(lens), len(picks))
    if values == "none":
        A.num = B.num = None
    plan = spx.GemmPlan(spx.from_host(A), spx.from_host(B), semiring)
    got, info = plan.execute().to_host_csc(), plan.info()
    plan.close()
    assert info["cols_tiny"] == len(picks)
    # each run of equal rows is summed in the oracle's order
    assert_same_csc(got, oracle.spgemm_csc(A, B, semiring, nthreads=1), exact_values=True, what=f"m={m} {semiring}")
