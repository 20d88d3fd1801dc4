"""SpRef at the edges of its column classes: outputs 64 | 512 | 4096, gathered
entries 256 | 4096, and the lengths of I past which keys take 64 bits or the
positions' ranks no longer come from a bitmap."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu

OUTPUTS = [0, 1, 63, 64, 65, 128, 129, 256, 257, 511, 512, 513, 4095, 4096, 4097]
GATHERED = [255, 256, 257, 4095, 4096, 4097, 9000]
SELECTED = 5000  # rows below this are in I


def matrix(sizes, m, values, seed):
    """One column per (gathered, outputs) of sizes: `outputs` rows below SELECTED, the rest above."""
    rng = np.random.default_rng(seed)
    rows = [np.concatenate([rng.choice(SELECTED, s, replace=False), SELECTED + rng.choice(m - SELECTED, g - s, replace=False)])
            for g, s in sizes]
    ir = np.concatenate(rows)
    num = None if values is None else np.arange(ir.size).astype(values)
    A = W.from_triples(ir, np.repeat(np.arange(len(sizes)), [r.size for r in rows]),
                       np.zeros(ir.size) if num is None else num, m, len(sizes))
    if num is None:
        A.num = None
    return A


def check(spx, A, I, J, real, what):
    """real: the positions of I whose rows A holds (the others select nothing), ascending."""
    B = spx.spref(spx.from_host(A), I, J).to_host_csc()
    ref = oracle.spref(A, I[real], J)
    ref.ir = real[ref.ir].astype(np.int32)
    assert_same_csc(B, ref, exact_values=True, what=what)


@pytest.mark.parametrize("values", ["i8", "f4", None])
@pytest.mark.parametrize("rep", [1, 2])  # times each selected row is in I
def test_class_edges(spx, values, rep):
    rng = np.random.default_rng(rep)
    sizes = [(max(s, 1) if s else 7, s) for s in OUTPUTS] + [(g, s) for g in GATHERED for s in (1, 64, 65) if s <= g]
    A = matrix(sizes, 20_000, values, seed=41)
    I = rng.permutation(np.repeat(np.arange(SELECTED), rep)).astype(np.int32)
    J = rng.permutation(np.concatenate([np.arange(A.n), rng.integers(0, A.n, 40)])).astype(np.int32)
    check(spx, A, I, J, np.arange(I.size), f"{values} x{rep}")


# lenI: 2^19 positions are ranked by bitmap, more by an LDS sort; past 2^23 the keys of
# up to 512 outputs take 64 bits, past 2^26 those of up to 64
@pytest.mark.parametrize("len_i", [(1 << 19) - 1, 1 << 19, (1 << 19) + 1, 1 << 23, (1 << 23) + 1, (1 << 26) + 5])
def test_long_index_vectors(spx, len_i):
    rng = np.random.default_rng(len_i % 97)
    sizes = [(max(s, 1), s) for s in OUTPUTS if 0 < s <= 4096] + [(9000, s) for s in (1, 40, 700)]
    A = matrix(sizes, 40_000, "i8", seed=43)
    m = 1 << 20
    A.m = m  # rows from 40000 on are empty
    I = (40_000 + np.arange(len_i, dtype=np.int64) % (m - 40_000)).astype(np.int32)
    real = np.unique(np.concatenate([[0, len_i - 1], rng.integers(0, len_i, 3 * SELECTED)]))
    real = np.sort(rng.choice(real, SELECTED, replace=False))
    I[real] = rng.permutation(SELECTED).astype(np.int32)
    J = rng.permutation(np.repeat(np.arange(A.n), 2)).astype(np.int32)
    check(spx, A, I, J, real, f"len(I)={len_i}")
