"""Stage sums of hypersparse blocks: offsets of the right blocks' columns found over
stored columns only, beside a stored-empty stage, a CSC one and columns shared by stages."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu

M, INNER = 300, 80


def stages(spx, n, kinds, seed):
    """Blocks A_k (M x INNER) and B_k (INNER x n): B_k of kinds[k] entries a column in
    some of 200 columns (the first and the last among them), negative: stored as CSC."""
    import torch
    rng = np.random.default_rng(seed)
    used = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 198)]))
    As = [W.erdos_renyi(M, INNER, 5, seed=seed + k, values="f64") for k in range(len(kinds))]
    Bs, dBs = [], []
    ids = torch.from_numpy(used.astype(np.int32)).cuda()
    for k, d in enumerate(kinds):
        cols = np.sort(rng.choice(used.size, used.size * 2 // 3, replace=False)) if k % 2 else np.arange(used.size)
        B = W.erdos_renyi(INNER, cols.size, abs(d), seed=seed + 50 + k, values="f64")
        B = W.from_triples(B.ir, np.repeat(cols, abs(d)), B.num, INNER, used.size)
        dB = spx.csc_to_dcsc(spx.from_host(B))
        dB.jc, dB.n = ids[dB.jc.long()], n
        Bs.append(B)
        dBs.append(spx.dcsc_to_csc(dB) if d < 0 else dB)
    return used, As, Bs, [spx.from_host(A) for A in As], dBs


@pytest.mark.parametrize("n,kinds", [
    ((1 << 20) + 7, [3, 0, 70, 1, 2, 80, 3, 5]),       # by stage
    ((1 << 20) + 7, [3, -2, 70] + [1] * 7),            # one CSC stage of ten: by stage
    ((1 << 20) + 7, [3, -2, 70]),                      # one of three: by table
    (1 << 20, [3, 0, 70, 1]),                          # short enough for the table
    ((1 << 24) - 1, [1, 2, 66]),
])
def test_hypersparse_stages(spx, n, kinds):
    used, As, Bs, dAs, dBs = stages(spx, n, kinds, seed=n % 1000 + len(kinds))
    ref = oracle.summa_stages(As, Bs, "plus_times")
    C = spx.spgemm_sum(dAs, dBs, out_fmt=spx.DCSC)
    slots = np.searchsorted(used, C.jc.cpu().numpy())
    assert np.array_equal(used[slots], C.jc.cpu().numpy())
    cp = np.zeros(used.size + 1, np.int64)
    cp[slots + 1] = np.diff(C.cp.cpu().numpy())
    got = W.from_triples([], [], np.empty(0), M, used.size)
    got.cp, got.ir, got.num = np.cumsum(cp), C.ir.cpu().numpy(), C.num.cpu().numpy()
    assert_same_csc(got, ref, what=f"n={n} {kinds}")


def test_memory_does_not_grow_with_stages_times_columns(spx):
    import torch
    n, peak = 1 << 22, []
    for count in (2, 10):
        used, As, Bs, dAs, dBs = stages(spx, n, [2] * count, seed=5)
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        spx.spgemm_sum(dAs, dBs, out_fmt=spx.DCSC)
        peak.append(torch.cuda.max_memory_allocated() - before)
    assert peak[1] - peak[0] < 4 * n, peak  # a word for each column and stage more would be 8 * 4 n
