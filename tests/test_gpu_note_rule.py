"""Heavy columns whose products per output lie on both sides of the line up to
which parts note a row with every product, whole and cut into parts."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,c", [(3000, 2000), (200_000, 60_000)])  # one part; several, over more than 65536 rows
@pytest.mark.parametrize("semiring,values", [("plus_times", "f8"), ("plus_times", "i8"), ("min_plus", "f4"),
                                             ("or_and", None)])
def test_products_per_output(spx, m, c, semiring, values):
    rng = np.random.default_rng(c)
    rows = np.sort(rng.choice(m, c, replace=False))  # of every column of A
    k = 40

    def num(n):
        return rng.integers(1, 9, n).astype(values or "f8")

    A = W.from_triples(np.tile(rows, k), np.repeat(np.arange(k), c), num(k * c), m, k)
    per = [15, 16, 17, 33, 1, 2]  # products of each output
    pick = np.concatenate([rng.choice(k, r, replace=False) for r in per])
    B = W.from_triples(pick, np.repeat(np.arange(len(per)), per), num(pick.size), k, len(per))
    if values is None:
        A.num = B.num = None
    plan = spx.GemmPlan(spx.from_host(A), spx.from_host(B), semiring)
    got, info = plan.execute().to_host_csc(), plan.info()
    plan.close()
    assert info["multi_parts"] >= len(per) and (info["multi_parts"] > len(per)) == (m > 65536)
    # sums of at most 33 products of whole numbers up to 64: exact in every type
    assert_same_csc(got, oracle.spgemm_csc(A, B, semiring, nthreads=8), exact_values=True, what=f"{semiring} m={m}")
