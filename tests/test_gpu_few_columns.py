"""Products of few columns, whose plans bin and scan the columns in one
workgroup, around the number of columns and of B's rows where that ends."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 1025, 8191, 8192, 8193])
@pytest.mark.parametrize("inner", [8192, 8193])
@pytest.mark.parametrize("dcsc", [False, True])
def test_few_columns(spx, n, inner, dcsc):
    rng = np.random.default_rng(n + inner)
    lens = rng.integers(0, 4, n)
    lens[rng.integers(0, n, 5)] = [300, 257, 256, 90, 2000]  # long columns, in every bin
    lens[-1] = 40
    rows = np.concatenate([np.sort(rng.choice(inner, d, replace=False)) for d in lens])
    B = W.from_triples(rows, np.repeat(np.arange(n), lens), rng.integers(1, 9, rows.size), inner, n)
    A = W.erdos_renyi(500, inner, 9, seed=7, values="f64")
    A.num = rng.integers(1, 9, A.ir.size).astype(np.int64)
    dA, dB = spx.from_host(A), spx.from_host(B)
    if dcsc:
        dA, dB = spx.csc_to_dcsc(dA), spx.csc_to_dcsc(dB)
    plan = spx.GemmPlan(dA, dB, "plus_times", spx.DCSC if dcsc else spx.CSC)
    got, info = plan.execute().to_host_csc(), plan.info()
    plan.close()
    ref = oracle.spgemm_csc(A, B, "plus_times")
    assert_same_csc(got, ref, exact_values=True, what=f"n={n} inner={inner}")
    mu, len_c = np.zeros(n, np.int64), np.diff(ref.cp)
    np.add.at(mu, np.repeat(np.arange(n), lens), 9)
    assert info["mults"] == mu.sum() and info["nnz"] == ref.cp[-1] and info["nzc"] == (len_c > 0).sum()
    assert info["cols_tiny"] == ((mu > 0) & (mu <= 64)).sum() and info["nnz_tiny"] == len_c[mu <= 64].sum()
