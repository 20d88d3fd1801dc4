"""Columns of 65 to 512 products (one wave each) at the edges of their register
classes: 64 | 65..128 | 129..256 | 257..512 | 513, against the CPU oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu

COUNTS = [1, 63, 64, 65, 66, 127, 128, 129, 130, 255, 256, 257, 300, 511, 512, 513]


def operands(m, values, seed):
    """A (m x 760): 520 columns of one row, 180 of seven, 60 empty ones, shuffled;
    B: one column per count of COUNTS, through short, longer and empty columns
    of A (more than 64 B entries for most counts)."""
    rng = np.random.default_rng(seed)
    kinds = rng.permutation(np.repeat([1, 7, 0], [520, 180, 60]))
    rows, cols = [], []
    for k, d in enumerate(kinds):
        rows.append(rng.choice(m, size=d, replace=False) if m < 10000 else np.unique(rng.integers(0, m, 4 * d + 1))[:d])
        cols.append(np.full(d, k))
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    ones, sevens, empty = (np.nonzero(kinds == d)[0] for d in (1, 7, 0))

    def vals(n):
        return rng.integers(1, 10, n) if values == "i64" else rng.random(n).astype(values)

    A = W.from_triples(rows, cols, vals(rows.size), m, kinds.size)
    bk, bj = [], []
    for j, mu in enumerate(COUNTS):
        s = min(mu // 14, 40)
        pick = np.concatenate([rng.permutation(sevens)[:s], rng.permutation(ones)[:mu - 7 * s], empty[:20]])
        bk.append(pick)
        bj.append(np.full(pick.size, j))
    bk, bj = np.concatenate(bk), np.concatenate(bj)
    return A, W.from_triples(bk, bj, vals(bk.size), kinds.size, len(COUNTS))


# 60 rows: every product meets others; 2^26 rows: (row, product) keys need 64 bits in every class
@pytest.mark.parametrize("m", [60, 5000, (1 << 23) + 1, 1 << 26])
@pytest.mark.parametrize("semiring,values", [("plus_times", "i64"), ("plus_times", "float64"), ("plus_times", "float32"),
                                             ("min_plus", "float64"), ("select2nd", "float32"), ("or_and", "i64")])
def test_mid_columns(spx, m, semiring, values):
    A, B = operands(m, values, seed=700 + m % 97)
    plan = spx.GemmPlan(spx.from_host(A), spx.from_host(B), semiring)
    got, info = plan.execute().to_host_csc(), plan.info()
    again = plan.execute().to_host_csc()
    plan.close()
    ref = oracle.spgemm_csc(A, B, semiring, nthreads=1)
    exact = not (semiring == "plus_times" and values != "i64")
    for g in (got, again):
        assert_same_csc(g, ref, exact_values=exact, what=f"{semiring} {values} m={m}")
    assert info["cols_medium"] == sum(mu > 64 for mu in COUNTS)
    assert info["heavy_parts"] >= info["cols_medium"]
