"""Bitmap counts in chunks of fewer rows than one 16-byte store takes: row blocks
of 64 rows (a small part budget) with chunks of 64 rows asked for, or row slices that short."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu


# 1024 rows: the last chunk ends where the next column's bitmap begins
@pytest.mark.parametrize("m", [100, 1000, 1024, 4096])
@pytest.mark.parametrize("semiring,values,lds", [("plus_times", "f64", 1024), ("min_plus", "f64", 1024),
                                                 ("plus_times", "f32", 600)])
@pytest.mark.parametrize("tune", [dict(bitmap_chunk_log2=6), dict(bitmap_chunk_log2=1), dict(bitmap_chunk_log2=7),
                                  dict(xcd_slices=64), dict(bitmap_chunk_log2=6, bitmap_store_mb=0)])
def test_short_bitmap_chunks(spx, m, semiring, values, lds, tune):
    A = W.erdos_renyi(m, 300, 8, seed=m, values=values)
    B = W.erdos_renyi(300, 70, 40, seed=m + 1, values=values)
    t = spx.default_tuning()
    for k, v in dict(tiny_max=0, hash_count_max=0, part_lds_bytes=lds, **tune).items():
        setattr(t, k, v)
    plan = spx.GemmPlan(spx.from_host(A), spx.from_host(B), semiring, tuning=t)
    got, info = plan.execute().to_host_csc(), plan.info()
    plan.close()
    assert info["cols_heavy"] == 70
    ref = oracle.spgemm_csc(A, B, semiring, nthreads=1)
    assert_same_csc(got, ref, exact_values=semiring == "min_plus", what=f"m={m} {tune}")
