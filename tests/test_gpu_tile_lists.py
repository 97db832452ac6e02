"""Shared lists of tiles (k_dist_topk's buffered selection and k_refine): the
ways a batch is split over the workgroups, ties, the parity-grouped INT8 order
and every list length, against the oracle bit for bit."""
import sys

import numpy as np
import pytest

import oracle
import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu

I8, F16, BF16, NB, FP8 = (L.LNBNN_EXACT_I8, L.LNBNN_EXACT_F16, L.LNBNN_EXACT_BF16, L.LNBNN_NBNN_I8,
                          L.LNBNN_FP8_RERANK)


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _check(got, want):
    cls, tot, ni, nd = got
    wt, wc, wi, wd = want
    assert np.array_equal(ni, wi) and np.array_equal(nd.astype(np.int64), wd)
    assert np.array_equal(tot, wt) and np.array_equal(cls, wc)


@pytest.fixture(scope="module")
def walk_set():
    # 64,013 references (2,001 tiles and more, ragged), 7 images
    rng = np.random.default_rng(71)
    R = rng.integers(0, 256, size=(64013, 128), dtype=np.uint8)
    labels = rng.integers(0, 9, size=R.shape[0]).astype(np.int32)
    Q = R[rng.integers(0, R.shape[0], size=6100)].copy()
    Q[::3] = rng.integers(0, 256, size=Q[::3].shape, dtype=np.uint8)
    off = np.array([0, 1, 600, 1700, 1700, 3100, 5000, 6100], np.int64)
    want = oracle.classify(Q, R, labels, 9, off, 10, route="block")
    ix = L.lnbnn_build_index(R, labels, 9, sum(L.LNBNN_MODE_BIT(m) for m in (I8, F16, NB)))
    yield R, labels, Q, off, ix, want
    ix.free()


@pytest.mark.parametrize("mode", [I8, F16, NB])
@pytest.mark.parametrize("workgroups,n_img", [
    (0, 7),      # 12 blocks of 512 queries on the whole GPU: slices
    (7, 7),      # one full round and 5 blocks: runs that cross block ends
    (5, 5),      # 7 blocks: a full round and 2 blocks in slices
    (12, 7),     # a full round exactly
    (1, 2),      # one workgroup
])
def test_walks(walk_set, mode, workgroups, n_img):
    R, labels, Q, off, ix, (wt, wc, wi, wd) = walk_set
    off = off[:n_img + 1]
    n = int(off[-1])
    for chunk in (0, 512):
        _say(f"walk mode={mode} workgroups={workgroups} images={n_img} chunk={chunk}")
        L.lnbnn_set_tuning(ix, mode, 10, chunk_tiles=chunk, max_workgroups=workgroups)
        try:
            got = L.lnbnn_classify(ix, Q[:n], off, 10, mode, want_neighbours=mode != NB)
        finally:
            L.lnbnn_set_tuning(ix, mode, 10)
        if mode == NB:
            _, _, D = oracle.knn_class_block(Q[:n], R, labels, 9, 1)
            tot, cls = oracle.nbnn(D, off)
            assert np.array_equal(got[1], tot) and np.array_equal(got[0], cls)
        else:
            _check(got, (wt[:n_img], wc[:n_img], wi[:n], wd[:n]))


@pytest.mark.parametrize("mode", [I8, NB])
@pytest.mark.parametrize("workgroups,chunk,n_img", [(0, 0, 7), (3, 512, 7), (4, 0, 6), (1, 8, 2), (0, 0, 1)])
def test_query_halves(walk_set, mode, workgroups, chunk, n_img):
    """Two query halves per wave (blocks of 1,024 queries): slices, runs, whole
    rounds with parked lists, a last block of a few queries, one query."""
    R, labels, Q, off, ix, (wt, wc, wi, wd) = walk_set
    off = off[:n_img + 1]
    n = int(off[-1])
    _say(f"halves mode={mode} workgroups={workgroups} chunk={chunk} images={n_img}")
    L.lnbnn_set_tuning(ix, mode, 10, variant=28, chunk_tiles=chunk, max_workgroups=workgroups)
    try:
        got = L.lnbnn_classify(ix, Q[:n], off, 10, mode, flags=L.LNBNN_TIMING, want_neighbours=mode != NB)
        assert L.lnbnn_last_timing(ix)["tile_variant"] == 28
    finally:
        L.lnbnn_set_tuning(ix, mode, 10)
    if mode == NB:
        _, _, D = oracle.knn_class_block(Q[:n], R, labels, 9, 1)
        tot, cls = oracle.nbnn(D, off)
        assert np.array_equal(got[1], tot) and np.array_equal(got[0], cls)
    else:
        _check(got, (wt[:n_img], wc[:n_img], wi[:n], wd[:n]))


@pytest.mark.parametrize("mode", [I8, F16, BF16])
@pytest.mark.parametrize("kind", ["ties", "even", "odd", "one_odd", "loc"])
def test_ties_and_parities(mode, kind):
    """Equal keys across tiles, lists and slices; indexes whose rows all have
    an even or an odd ||r - 128||^2, or all but one."""
    if kind == "loc" and mode != I8:
        pytest.skip("160-byte rows: INT8 only")
    rng = np.random.default_rng(5)
    dim = 160 if kind == "loc" else 128
    n = 5001
    R = rng.integers(0, 2, size=(n, dim), dtype=np.uint8)
    R[:, 3:] = R[:, 3:4]                     # few distinct rows: ties everywhere
    if kind in ("even", "odd", "one_odd"):
        R = rng.integers(0, 256, size=(n, dim), dtype=np.uint8)
        odd = R.astype(np.int64).sum(1) % 2
        R[:, 0] ^= (odd != (kind == "odd")).astype(np.uint8)
        if kind == "one_odd":
            R[4321, 0] ^= 1
    labels = rng.integers(0, 6, size=n).astype(np.int32)
    Q = R[rng.integers(0, n, size=150)].copy()
    Q[::2, 1] ^= 1
    off = np.array([0, 40, 40, 150], np.int64)
    ix = L.lnbnn_build_index(R, labels, 6, L.LNBNN_MODE_BIT(mode))
    try:
        for k in (1, 5, 10, 15, 20, 32):
            _say(f"{kind} mode={mode} k={k}")
            got = L.lnbnn_classify(ix, Q, off, k, mode, want_neighbours=True)
            _check(got, oracle.classify(Q, R, labels, 6, off, k))
    finally:
        ix.free()


@pytest.mark.parametrize("k", [1, 2, 5, 10, 11, 16])
def test_fp8_candidates_do_not_depend_on_the_walk(k):
    """The FP8 top 4k by (key, index) is defined without the launch plan:
    every split, and the row-wise per-half lists (variant 0), give the same
    bits."""
    rng = np.random.default_rng(9)
    R = np.maximum(rng.standard_normal((40007, 128)), 0).astype(np.float32)
    R[::50] = R[7]                           # equal keys
    labels = rng.integers(0, 12, size=R.shape[0]).astype(np.int32)
    Q = np.maximum(R[rng.integers(0, R.shape[0], size=1300)] + 0.1 * rng.standard_normal((1300, 128)), 0)
    Q = Q.astype(np.float32)
    off = np.array([0, 300, 1300], np.int64)
    ix = L.lnbnn_build_index(R, labels, 12, L.LNBNN_MODE_BIT(FP8))
    try:
        L.lnbnn_set_tuning(ix, FP8, k, variant=0)
        want = L.lnbnn_classify(ix, Q, off, k, FP8, want_neighbours=True)
        for workgroups in (0, 1, 2, 5):
            _say(f"fp8 k={k} workgroups={workgroups}")
            L.lnbnn_set_tuning(ix, FP8, k, max_workgroups=workgroups)
            got = L.lnbnn_classify(ix, Q, off, k, FP8, want_neighbours=True)
            for x, y in zip(want, got):
                assert np.array_equal(x, y)
    finally:
        ix.free()


@pytest.mark.parametrize("n_ref,n_q,workgroups,k,want,other", [
    (131063, 1300, 1, 1, 8, 11),    # 4,096 tiles in one slice
    (131063, 1300, 1, 3, 8, 11),
    (131063, 1300, 1, 5, 11, 8),    # lists of 20
    (786401, 700, 1, 5, 8, 11),     # 24,576 tiles
    (130711, 1300, 1, 1, 11, 8),    # 4,085 tiles, fewer items than CUs
    (64013, 4096, 0, 1, 8, 8),      # 8 blocks of 512 in 32 slices: 256 items
    (64013, 4096, 0, 2, 8, 8),
])
def test_union_of_halves_shapes(n_ref, n_q, workgroups, k, want, other):
    """Default shape of the union-of-halves FP8 rule: where the slices are the
    same, so are the lists, and every result is equal to the other shape's."""
    rng = np.random.default_rng(n_ref + k)
    R = rng.standard_normal((n_ref, 128), dtype=np.float32)
    labels = rng.integers(0, 5, size=n_ref).astype(np.int32)
    Q = rng.standard_normal((n_q, 128), dtype=np.float32)
    off = np.array([0, 1, 700, n_q], np.int64)
    mode = L.LNBNN_FP8_RERANK_2K
    ix = L.lnbnn_build_index(R, labels, 5, L.LNBNN_MODE_BIT(mode))
    try:
        res = []
        for v in (-1, other):
            _say(f"union refs={n_ref} queries={n_q} workgroups={workgroups} k={k} variant={v}")
            L.lnbnn_set_tuning(ix, mode, k, variant=v, max_workgroups=workgroups)
            res.append(L.lnbnn_classify(ix, Q, off, k, mode, flags=L.LNBNN_TIMING, want_neighbours=True))
            assert L.lnbnn_last_timing(ix)["tile_variant"] == (want if v < 0 else other)
    finally:
        ix.free()
    for a, b in zip(*res):
        assert np.array_equal(a, b)
