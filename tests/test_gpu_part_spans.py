"""Row-range parts that fill up by their span, not by their outputs: hash parts of
up to 2^20 rows, whose rows a bitmap ranks, longer ones, whose rows are sorted, and
bitmap parts over more than 65536 rows, whose noted rows need their high bits."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu

KINDS = [("plus_times", "f8"), ("plus_times", "i8"), ("min_plus", "f4"), ("or_and", None)]


def product(spx, m, per_a, ncols_a, per, cols, semiring, values, seed, last_row=True):
    rng = np.random.default_rng(seed)
    rows = [np.unique(rng.integers(0, m, per_a)) for _ in range(ncols_a)]
    if last_row:
        for r in rows:
            r[-1] = m - 1

    def num(n):
        return rng.integers(1, 9, n).astype(values or "f8")  # small whole numbers: every sum is exact

    lens = [r.size for r in rows]
    A = W.from_triples(np.concatenate(rows), np.repeat(np.arange(ncols_a), lens), num(sum(lens)), m, ncols_a)
    k = np.concatenate([np.sort(rng.choice(ncols_a, per, replace=False)) for _ in range(cols)])
    B = W.from_triples(k, np.repeat(np.arange(cols), per), num(k.size), ncols_a, cols)
    if values is None:
        A.num = B.num = None
    plan = spx.GemmPlan(spx.from_host(A), spx.from_host(B), semiring)
    got, info = plan.execute().to_host_csc(), plan.info()
    plan.close()
    ref = oracle.spgemm_csc(A, B, semiring, nthreads=8)
    assert_same_csc(got, ref, exact_values=True, what=f"m={m} {semiring} {values}")
    return ref, info


# 2000 products a column, one hash part's worth: cut where 2^20 rows end while that makes
# at most three parts.  5000 products, three parts' worth: while it makes at most nine.
@pytest.mark.parametrize("m,per_a,cut", [(1 << 20, 500, True), ((1 << 20) + 1, 500, True), (3 << 20, 500, True),
                                         ((3 << 20) + 1, 500, False), ((1 << 24) + 77, 500, False),
                                         (9 << 20, 1250, True), ((9 << 20) + 1, 1250, False)])
@pytest.mark.parametrize("semiring,values", KINDS)
def test_hash_part_spans(spx, m, per_a, cut, semiring, values):
    cols = 12
    ref, info = product(spx, m, per_a, 8, 4, cols, semiring, values, seed=m % 1013)
    outputs = np.diff(ref.cp)
    need = -(-4 * per_a // 2048)
    assert outputs.min() > max(1024, 2048 * (need - 1)) and outputs.max() <= 2048 * need
    spans = np.unique(np.repeat(np.arange(cols), outputs) * 64 + (ref.ir >> 20)).size
    assert info["multi_parts"] == (spans if cut else need * cols)


# 5400 products over 500000 rows: two bitmap parts of 250000 rows or more to a column.
# Every product's row is noted in all parts of many columns, and in a column's last part of few.
@pytest.mark.parametrize("cols", [4200, 40])
@pytest.mark.parametrize("semiring,values", KINDS)
def test_noted_rows_past_65536(spx, cols, semiring, values):
    ref, info = product(spx, 500_000, 1800, 40, 3, cols, semiring, values, seed=cols)
    assert np.diff(ref.cp).min() > 5000
    assert info["multi_parts"] == 2 * cols
