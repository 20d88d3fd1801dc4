"""How the row-range parts of heavy columns are accumulated and written: rows
noted per product (many cut columns), hash parts cut at the span whose rows
they rank by bitmap, and hash parts of wider spans, which sort their rows."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu

CASES = {
    # 4200 columns of 12000 products in two parts or more, some rows met up to three times
    "noted_rows": dict(m=60_000, a=[4000] * 40, cols=4200, per=3),
    # outputs spread over three spans of 2^20 rows; 2000 to 9000 outputs a part
    "ranked_spans": dict(m=3 << 20, a=[3000] * 6 + [12_000, 700, 40], cols=12, per=4),
    # rows past four such spans, the last part short
    "wide_spans": dict(m=(4 << 20) + 77, a=[3000] * 6 + [9000, 500], cols=10, per=5),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("semiring,values", [("plus_times", "f64"), ("min_plus", "f32"), ("or_and", "none")])
def test_parts(spx, name, semiring, values):
    c = CASES[name]
    rng = np.random.default_rng(len(name))

    def num(n):
        return rng.random(n).astype("f4" if values == "f32" else "f8")

    rows = [np.unique(rng.integers(0, c["m"], d)) for d in c["a"]]
    rows[0][-1] = c["m"] - 1
    lens = [r.size for r in rows]
    A = W.from_triples(np.concatenate(rows), np.repeat(np.arange(len(rows)), lens), num(sum(lens)), c["m"], len(rows))
    k = np.concatenate([np.sort(rng.choice(len(rows), c["per"], replace=False)) for _ in range(c["cols"])])
    B = W.from_triples(k, np.repeat(np.arange(c["cols"]), c["per"]), num(k.size), len(rows), c["cols"])
    if values == "none":
        A.num = B.num = None
    got = spx.spgemm(spx.from_host(A), spx.from_host(B), semiring).to_host_csc()
    ref = oracle.spgemm_csc(A, B, semiring, nthreads=8)
    assert_same_csc(got, ref, exact_values=values != "f64", what=f"{name} {semiring}")
