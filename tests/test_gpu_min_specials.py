"""(min,+), select1st and select2nd over NaN, infinities and signed zeros in
columns of 65 to 512 products, whose runs of equal rows are folded in pieces:
NaN is passed over (a row of NaN alone gives +inf) and -0 is less than +0,
wherever in the run they lie, as in the wider columns that use LDS minima."""
import warnings

import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

COUNTS = [66, 128, 130, 256, 258, 300, 512]  # products of each column, in every register class


def operands(rows, val, first, seed):
    """A (rows x 512, full columns) and B, whose column j has COUNTS[j] // rows
    entries.  Column 0 of A and row 0 of B, which give each row's first product,
    hold no NaN if first is "number"; of the rest a third is NaN."""
    rng = np.random.default_rng(seed)

    def vals(n, k):
        v = rng.choice(np.array([-3, -1, -0.0, 0.0, 0.0, 2, 5, np.inf, -np.inf]), n).astype(val)
        v[rng.random(n) < 1 / 3] = np.nan
        if first == "number":
            v[k == 0] = rng.choice(np.array([0.0, 4, np.inf]), (k == 0).sum())
        return v

    ka = np.repeat(np.arange(512), rows)
    A = W.from_triples(np.tile(np.arange(rows), 512), ka, vals(ka.size, ka), rows, 512)
    kb = [np.concatenate([[0], rng.choice(np.arange(1, 512), mu // rows - 1, replace=False)]) for mu in COUNTS]
    jb = np.repeat(np.arange(len(COUNTS)), [k.size for k in kb])
    kb = np.concatenate(kb)
    return A, W.from_triples(kb, jb, vals(kb.size, kb), 512, len(COUNTS))


@pytest.mark.parametrize("rows", [1, 2, 7, 33])  # runs through the whole wave, several lanes, one lane
@pytest.mark.parametrize("semiring", ["min_plus", "select1st", "select2nd"])
@pytest.mark.parametrize("val", ["f4", "f8"])
def test_min_passes_over_nan(spx, rows, semiring, val):
    for first in ("number", "any"):
        A, B = operands(rows, val, first, 31 * rows + (first == "any"))
        got = spx.spgemm(spx.from_host(A), spx.from_host(B), semiring).to_host_csc()
        ref = oracle.spgemm_csc(A, B, semiring, nthreads=1).num
        a = A.num.reshape(512, rows)
        want = []
        for j in range(B.n):
            k, b = B.ir[B.cp[j]:B.cp[j + 1]], B.num[B.cp[j]:B.cp[j + 1]]
            if k.size * rows <= 64:  # 9 of 7 rows: a tiny column, which Algorithm 1 folds
                want.append(ref[j * rows:(j + 1) * rows])
                continue
            with warnings.catch_warnings():
                warnings.simplefilter("ignore")  # inf - inf
                x = a[k] + b[:, None] if semiring == "min_plus" else a[k] if semiring == "select1st" else \
                    np.broadcast_to(b[:, None], (k.size, rows))
            low = np.where(np.isnan(x), np.inf, x).min(0)
            minus = ((x == 0) & np.signbit(x)).any(0)
            want.append(np.where(low == 0, np.where(minus, -0.0, 0.0), low).astype(val))
        want = np.concatenate(want)
        bits = {"f4": np.uint32, "f8": np.uint64}[val]
        bad = np.nonzero((got.num.view(bits) != want.view(bits)) & ~(np.isnan(got.num) & np.isnan(want)))[0]
        assert bad.size == 0, f"{semiring} {first}: {bad.size} differ, {got.num[bad[:5]]} for {want[bad[:5]]}"
        if first == "number":  # Algorithm 1, up to the sign of zeros
            assert np.array_equal(got.num, ref)
