"""SpAsgn around the 1024-entry tiles and the 2048-column blocks: modified columns
inside one tile, across several, ending on their edges, and column pointers
where the number of columns ends a block."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import assert_same_csc

pytestmark = pytest.mark.gpu


def _matrix(rng, m, lens):
    rows = np.concatenate([np.sort(rng.choice(m, d, replace=False)) for d in lens]) if sum(lens) else np.empty(0, np.int64)
    A = W.from_triples(rows, np.repeat(np.arange(len(lens)), lens), np.arange(rows.size, dtype=np.int64), m, len(lens))
    return A


@pytest.mark.parametrize("picked", ["none", "first", "last", "every", "some"])
@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 4096])
def test_columns_around_blocks(spx, n, picked):
    rng = np.random.default_rng(n)
    A = _matrix(rng, 90, rng.integers(0, 5, n))
    J = {"none": [], "first": [0], "last": [n - 1], "every": rng.permutation(n), "some": rng.integers(0, n, 40)}[picked]
    J, I = np.asarray(J, np.int32), rng.integers(0, 90, 30).astype(np.int32)
    B = _matrix(rng, 30, rng.integers(0, 6, J.size)) if J.size else W.from_triples([], [], np.empty(0, np.int64), 30, 0)
    got = spx.spasgn(spx.from_host(A), I, J, spx.from_host(B)).to_host_csc()
    assert_same_csc(got, oracle.spasgn(A, I, J, B), exact_values=True, what=f"{n} {picked}")


@pytest.mark.parametrize("lens", [[1024], [1023], [1025], [1022, 1, 1024, 2], [5000], [0, 3000, 0, 3, 2200, 1024],
                                  [500] * 9, [16, 17] * 200, [1] * 3000])
@pytest.mark.parametrize("picked", ["every", "odd", "last"])
def test_columns_around_tiles(spx, lens, picked):
    rng = np.random.default_rng(sum(lens))
    A = _matrix(rng, 6000, lens)
    n = len(lens)
    J = np.asarray({"every": np.arange(n), "odd": np.arange(n)[::-2], "last": [n - 1]}[picked], np.int32)
    I = rng.permutation(6000)[:3500].astype(np.int32)
    B = _matrix(rng, 3500, rng.integers(0, 9, J.size))
    got = spx.spasgn(spx.from_host(A), I, J, spx.from_host(B)).to_host_csc()
    assert_same_csc(got, oracle.spasgn(A, I, J, B), exact_values=True, what=f"{lens[:6]} {picked}")


@pytest.mark.parametrize("picked", ["none", "first", "last", "every", "some"])
@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 4096])
def test_extend_add_around_blocks(spx, n, picked):
    rng = np.random.default_rng(n)
    lens = rng.integers(0, 5, n)
    lens[n // 2] = 1500  # an A column over tiles, and past the column kernels
    A = _matrix(rng, 1600, lens)
    J = {"none": [], "first": [0], "last": [n - 1] * 3, "every": rng.permutation(n), "some": rng.integers(0, n, 40)}[picked]
    J, I = np.asarray(J, np.int32), rng.integers(0, 1600, 90).astype(np.int32)
    B = _matrix(rng, 90, rng.integers(0, 80 if picked == "some" else 6, J.size)) if J.size \
        else W.from_triples([], [], np.empty(0, np.int64), 90, 0)
    got = spx.extend_add(spx.from_host(A), I, J, spx.from_host(B)).to_host_csc()
    assert_same_csc(got, oracle.extend_add(A, I, J, B), exact_values=True, what=f"{n} {picked}")
