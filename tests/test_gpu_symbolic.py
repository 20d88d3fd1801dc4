"""Branches of the SpGEMM plan (split table, hash counts in one or several
launches, part cutting) on products small enough for the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu


def with_columns(rng, m, lengths, val):
    """m x len(lengths) matrix whose column k holds lengths[k] distinct rows."""
    rows = [np.sort(rng.choice(m, d, replace=False)) if d * 4 > m else np.unique(rng.integers(0, m, 2 * d + 8))[:d]
            for d in lengths]
    rows = [r if r.size == d else np.sort(rng.choice(m, d, replace=False)) for r, d in zip(rows, lengths)]
    cols = np.repeat(np.arange(len(lengths)), lengths)
    rows = np.concatenate(rows)
    return W.from_triples(rows, cols, val(rows.size), m, len(lengths))


CASES = {
    # every column cut into parts; one A column of 19000 rows (searched split row); flat split notes
    "searched_split_row": dict(m=20000, a=[19000, 64, 33, 32, 900, 0, 7000], picks=[[0, 1, 2, 3, 4, 5, 6], [0, 6], [1, 4, 6]]),
    # more than 1024 row blocks: parts cut from memory instead of LDS
    "many_row_blocks": dict(m=9_500_000, a=[3000, 40, 2500, 35, 12, 4000], picks=[[0, 1, 2, 3, 4, 5], [0, 2, 5], [2, 3]]),
    # few cut columns among many (grouped split notes), one with more than 256 B entries
    "few_cut_columns": dict(m=6000, a=[40] * 300 + [3000, 2500], picks=[list(range(302)), [300, 301], [5]], pad=4000),
    # 513 to 8192 products: 600 columns in one hash launch, 1500 in one per table size
    "hash_together": dict(m=5000, a=[150] * 8 + [700] * 6, picks=[[0, 1, 2, 3, 4 + i % 4, 8 + i % 6] for i in range(600)]),
    "hash_apart": dict(m=5000, a=[150] * 8 + [700] * 6,
                       picks=[[0, 1, 2, 3, 4 + i % 4] + [8 + i % 6] * (i % 3 > 0) + [8 + (i + 1) % 6] * (i % 3 > 1)
                              for i in range(1500)]),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("semiring,values,a_dcsc", [("plus_times", "f64", False), ("plus_times", "i64", True),
                                                    ("min_plus", "f32", False)])
def test_plan_branches(spx, name, semiring, values, a_dcsc):
    c = CASES[name]
    rng = np.random.default_rng(len(name) * 31 + len(values))

    def val(n):
        return rng.integers(1, 10, n) if values == "i64" else rng.random(n).astype("f8" if values == "f64" else "f4")

    A = with_columns(rng, c["m"], c["a"], val)
    picks = [sorted(set(p)) for p in c["picks"]] + [[]] * c.get("pad", 0)
    k = np.concatenate([np.asarray(p, dtype=np.int64) for p in picks])
    B = W.from_triples(k, np.repeat(np.arange(len(picks)), [len(p) for p in picks]), val(k.size), A.n, len(picks))
    dA = spx.from_host(A)
    plan = spx.GemmPlan(spx.csc_to_dcsc(dA) if a_dcsc else dA, spx.from_host(B), semiring)
    got, info = plan.execute().to_host_csc(), plan.info()
    plan.close()
    ref = oracle.spgemm_csc(A, B, semiring, nthreads=1)
    assert_same_csc(got, ref, exact_values=values != "f64", what=f"{name} {semiring}")
    assert info["mults"] == int(np.diff(A.cp)[B.ir].sum()) and info["nnz"] == ref.cp[-1]
    assert info["nzc"] == int((np.diff(ref.cp) > 0).sum())
