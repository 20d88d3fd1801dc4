"""An exec that fails after its first launches leaves a plan that can run again."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu


def hip_runtime():
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    assert len(paths) == 1, paths
    return ctypes.CDLL(paths.pop())


@pytest.mark.parametrize("semiring", ["plus_times", "min_plus"])
def test_exec_after_failed_exec(spx, semiring):
    import torch
    A = W.rmat(13, 8, seed=3)  # cut columns, whole parts and tiny ones
    plan = spx.GemmPlan(spx.from_host(A), spx.from_host(A), semiring)
    info = plan.info()
    assert info["multi_parts"] > 0 and info["heavy_parts"] > info["multi_parts"]
    ref = oracle.spgemm_csc(A, A, semiring, nthreads=8)
    C = plan.alloc_output()
    hip = hip_runtime()
    torch.cuda.synchronize()
    # an error of another call that nobody has read is reported by the exec's first check
    assert hip.hipSetDevice(ctypes.c_int(1 << 20)) != 0
    with pytest.raises(spx.SpxError):
        plan.execute(C)
    torch.cuda.synchronize()
    for _ in range(2):
        C.ir.fill_(-1)
        C.num.fill_(-1)
        plan.execute(C)
        assert_same_csc(C.to_host_csc(), ref, exact_values=semiring == "min_plus", what=f"after a failed exec, {semiring}")
    plan.close()
