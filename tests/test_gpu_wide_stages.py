"""Stage sums whose right blocks have so many columns that their lengths are
tabled for one or two stages at a time."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1 << 25) - 5, (1 << 26) + 3])  # two stages at a time (of three), one at a time
def test_stage_sum_over_stage_groups(spx, n):
    import torch
    rng = np.random.default_rng(n)
    used = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 300)]))
    # 90 entries a column: placed by whole waves, 3: by 16 lanes
    As = [W.erdos_renyi(500, 100, 6, seed=k, values="f64") for k in range(3)]
    Bs = [W.erdos_renyi(100, used.size, (3, 0, 90)[k], seed=9 + k, values="f64") for k in range(3)]
    ref = oracle.summa_stages(As, Bs, "plus_times")
    ids = torch.from_numpy(used.astype(np.int32)).cuda()
    dBs = []
    for B in Bs:  # the same columns, spread over n
        d = spx.csc_to_dcsc(spx.from_host(B))
        d.jc, d.n = ids[d.jc.long()], n
        dBs.append(d)
    C = spx.spgemm_sum([spx.from_host(A) for A in As], dBs, out_fmt=spx.DCSC)
    slots = np.searchsorted(used, C.jc.cpu().numpy())
    assert np.array_equal(used[slots], C.jc.cpu().numpy())
    cp = np.zeros(used.size + 1, np.int64)
    cp[slots + 1] = np.diff(C.cp.cpu().numpy()[:slots.size + 1])
    got = W.from_triples([], [], np.empty(0), 500, used.size)
    got.cp, got.ir, got.num = np.cumsum(cp), C.ir.cpu().numpy()[:C.nnz], C.num.cpu().numpy()[:C.nnz]
    assert_same_csc(got, ref, what=f"stage groups, n={n}")
