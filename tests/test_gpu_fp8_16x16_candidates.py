"""The FP8 top-4k rule on 16x16 blocks (variants 25 and 27): the rows of a
query's best tiles are recomputed with the arithmetic that made the lists, so no
candidate is lost to the last place in which the two block shapes' keys differ."""
import sys

import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu
FP8 = L.LNBNN_FP8_RERANK


def _wide(rng, n):
    """Elements over fourteen powers of two, so that the sums behind the keys do not
    fit 24 bits and their rounding shows."""
    x = np.abs(rng.standard_normal((n, 128))) * 2.0 ** rng.uniform(-14, 0, (n, 128))
    return x.astype(np.float32)


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("variant", [25, 27])
@pytest.mark.parametrize("k", [1, 5, 10])
def test_repeated_rows_keep_their_candidates(variant, k):
    """Every row stands in more tiles than a list holds, so for a query next to
    it all the listed tiles have one smallest key, in either arithmetic, and the
    4k candidates are the row's first copies: the results are those of the
    row-wise lists (variant 0), bit for bit, for every split of the batch."""
    rng = np.random.default_rng(31)
    base = _wide(rng, 64)
    R = np.tile(base, (100, 1))
    labels = rng.integers(0, 12, size=R.shape[0]).astype(np.int32)
    at = rng.integers(0, 64, size=1500)
    Q = (base[at] * (1 + 0.05 * rng.standard_normal((1500, 128)))).astype(np.float32)
    off = np.array([0, 200, 200, 1500], np.int64)
    ix = L.lnbnn_build_index(R, labels, 12, L.LNBNN_MODE_BIT(FP8))
    try:
        L.lnbnn_set_tuning(ix, FP8, k, variant=0)
        want = L.lnbnn_classify(ix, Q, off, k, FP8, want_neighbours=True)
        assert np.array_equal(want[2], at[:, None] + 64 * np.arange(k + 1)[None, :])
        for chunk, workgroups in ((0, 0), (0, 1), (8, 2)):
            _say(f"fp8 repeated rows k={k} variant={variant} chunk={chunk} workgroups={workgroups}")
            L.lnbnn_set_tuning(ix, FP8, k, variant=variant, chunk_tiles=chunk, max_workgroups=workgroups)
            got = L.lnbnn_classify(ix, Q, off, k, FP8, want_neighbours=True)
            for x, y in zip(want, got):
                assert np.array_equal(x, y)
    finally:
        ix.free()


@pytest.mark.parametrize("k", [1, 2, 5, 10])
def test_candidates_do_not_depend_on_the_walk(k):
    """The 4k best rows by the 16x16 form's (key, index): both variants of it,
    and every split, give the same bits, with repeated rows among others."""
    rng = np.random.default_rng(32)
    R = _wide(rng, 40007)
    R[::50] = R[7]
    labels = rng.integers(0, 12, size=R.shape[0]).astype(np.int32)
    Q = R[rng.integers(0, R.shape[0], size=1300)] * (1 + 0.1 * rng.standard_normal((1300, 128)))
    Q = Q.astype(np.float32)
    off = np.array([0, 300, 1300], np.int64)
    ix = L.lnbnn_build_index(R, labels, 12, L.LNBNN_MODE_BIT(FP8))
    try:
        want = None
        for variant in (25, 27):
            for chunk, workgroups in ((0, 0), (0, 1), (0, 5), (8, 2)):
                _say(f"fp8 16x16 k={k} variant={variant} chunk={chunk} workgroups={workgroups}")
                L.lnbnn_set_tuning(ix, FP8, k, variant=variant, chunk_tiles=chunk, max_workgroups=workgroups)
                got = L.lnbnn_classify(ix, Q, off, k, FP8, want_neighbours=True)
                assert got[2].min() >= 0 and got[2].max() < R.shape[0]
                want = want or got
                for x, y in zip(want, got):
                    assert np.array_equal(x, y)
    finally:
        ix.free()


@pytest.mark.parametrize("n_refs,k", [(40, 10), (12, 3), (130, 10), (1003, 10)])
def test_small_indexes(n_refs, k):
    """Fewer tiles than the list holds (the pass without a bound), and 4k =
    n_refs, where every row is a candidate."""
    rng = np.random.default_rng(n_refs)
    R = np.maximum(rng.standard_normal((n_refs, 128)), 0).astype(np.float32)
    labels = rng.integers(0, 5, size=n_refs).astype(np.int32)
    Q = np.maximum(rng.standard_normal((150, 128)), 0).astype(np.float32)
    off = np.array([0, 70, 150], np.int64)
    ix = L.lnbnn_build_index(R, labels, 5, L.LNBNN_MODE_BIT(FP8))
    try:
        res = []
        for variant in (25, 27):
            L.lnbnn_set_tuning(ix, FP8, k, variant=variant)
            res.append(L.lnbnn_classify(ix, Q, off, k, FP8, want_neighbours=True))
            assert res[-1][2].min() >= 0 and res[-1][2].max() < n_refs
        if 4 * k == n_refs:
            L.lnbnn_set_tuning(ix, FP8, k, variant=0)
            res.append(L.lnbnn_classify(ix, Q, off, k, FP8, want_neighbours=True))
    finally:
        ix.free()
    for r in res[1:]:
        for x, y in zip(res[0], r):
            assert np.array_equal(x, y)
