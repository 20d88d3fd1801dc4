"""Plan statistics are known once the plan is made: asking for them launches
nothing and changes nothing, so it works during a capture and from several threads."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [13, 8])
def test_info_during_capture_and_from_threads(spx, scale):
    import torch
    A = W.rmat(scale, 8, seed=6)
    ref = oracle.spgemm_csc(A, A, nthreads=8)
    mults = np.add.reduceat(np.append(np.diff(A.cp)[A.ir], 0), A.cp[:-1]) * (np.diff(A.cp) > 0)
    cut = int(np.diff(ref.cp)[mults > 1024].sum())  # columns above single_part_max
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        plan = spx.GemmPlan(spx.from_host(A), spx.from_host(A))
    s.synchronize()
    x = torch.zeros(4, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        captured = plan.info()
        x.add_(1)
    with ThreadPoolExecutor(8) as ex:
        infos = list(ex.map(lambda _: plan.info(), range(64)))
    assert all(i == captured for i in infos)
    assert captured["nnz_multi"] == cut and captured["multi_parts"] > 0
    assert captured["nnz"] == ref.ir.size and captured["mults"] == mults.sum()
    for k in range(2):
        g.replay()
        torch.cuda.synchronize()
        assert x.tolist() == [k + 1.0] * 4
    plan.close()


# columns cut into row ranges: more products than single_part_max (512 at least), or than
# the hash count takes; a plan of up to 8192 columns and one of more
@pytest.mark.parametrize("scale", [12, 14])
@pytest.mark.parametrize("tune,above", [({}, 1024), (dict(single_part_max=2048), 2048), (dict(single_part_max=64), 512),
                                        (dict(hash_count_max=700), 700),
                                        (dict(tiny_max=0, hash_count_max=0), 0)])
def test_entries_of_cut_columns(spx, scale, tune, above):
    A = W.rmat(scale, 8, seed=7)
    ref = oracle.spgemm_csc(A, A, nthreads=8)
    mults = np.add.reduceat(np.append(np.diff(A.cp)[A.ir], 0), A.cp[:-1]) * (np.diff(A.cp) > 0)
    t = spx.default_tuning()
    for k, v in tune.items():
        setattr(t, k, v)
    plan = spx.GemmPlan(spx.from_host(A), spx.from_host(A), tuning=t)
    info = plan.info()
    plan.close()
    assert info["nnz_multi"] == np.diff(ref.cp)[mults > above].sum()
    assert info["nnz_tiny"] == np.diff(ref.cp)[mults <= t.tiny_max].sum()
