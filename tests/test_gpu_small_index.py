"""Exact searches of small indexes: how a batch is split and which lists it keeps,
on both sides of the rules, and the same results as the other shapes and as the
oracle, bit for bit."""
import sys

import numpy as np
import pytest

import oracle
import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu

I8, F16, BF16, NB = L.LNBNN_EXACT_I8, L.LNBNN_EXACT_F16, L.LNBNN_EXACT_BF16, L.LNBNN_NBNN_I8


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _set(n_refs, n_q, dim=128, classes=7):
    rng = np.random.default_rng(n_refs + n_q)
    R = rng.integers(0, 256, size=(n_refs, dim), dtype=np.uint8)
    R[::9] = R[3]                                  # ties
    labels = (np.arange(n_refs) % classes).astype(np.int32)
    Q = R[rng.integers(0, n_refs, size=n_q)].copy()
    Q[::3] = rng.integers(0, 256, size=Q[::3].shape, dtype=np.uint8)
    off = np.array([0, n_q // 3, n_q // 3, n_q], np.int64)
    return R, labels, Q, off


def _check_head(got, R, labels, Q, k):
    head = min(300, len(Q))
    wt, wc, wi, wd = oracle.classify(Q[:head], R, labels, int(labels.max()) + 1, np.array([0, head], np.int64), k)
    assert np.array_equal(got[2][:head], wi) and np.array_equal(got[3][:head].astype(np.int64), wd)


@pytest.mark.parametrize("mode,n_refs,n_q,k,cut", [
    (F16, 3000, 2000, 10, True),      # 4 blocks, 96 tiles: nothing but list start
    (I8, 3000, 2000, 5, True),
    (BF16, 2001, 16384, 10, True),    # 32 blocks: the last size with an eighth of the grid
    (F16, 2001, 16385, 10, False),    # 33 blocks
    (I8, 257, 1, 1, False),           # 16 tiles
    (NB, 12000, 100_000, 1, True),    # 98 blocks of 1,024, about 400 tiles
])
def test_short_sweeps_are_cut(mode, n_refs, n_q, k, cut):
    R, labels, Q, off = _set(n_refs, n_q)
    ix = L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode))
    nbr = mode != NB
    try:
        _say(f"cut mode={mode} refs={n_refs} queries={n_q} k={k}")
        got = L.lnbnn_classify(ix, Q, off, k, mode, flags=L.LNBNN_TIMING, want_neighbours=nbr)
        t = L.lnbnn_last_timing(ix)
        L.lnbnn_set_tuning(ix, mode, k, variant=t["tile_variant"], max_workgroups=1)   # whole sweeps
        want = L.lnbnn_classify(ix, Q, off, k, mode, flags=L.LNBNN_TIMING, want_neighbours=nbr)
        assert L.lnbnn_last_timing(ix)["slices"] == 1
    finally:
        ix.free()
    assert (t["slices"] > 1) == cut
    for x, y in zip(want, got):
        assert x is None or np.array_equal(x, y)
    if nbr:
        _check_head(got, R, labels, Q, k)


@pytest.mark.parametrize("n_refs,variant", [(7 * 80, 15), (7 * 300, 28)])
def test_algorithm_1_on_few_tiles(n_refs, variant):
    """Fewer than 64 tiles (14 groups of 256 rows are 112, two of them 16)."""
    classes = 2 if variant == 15 else 7
    R, labels, Q, off = _set(n_refs, 50_000, classes=classes)
    ix = L.lnbnn_build_index(R, labels, classes, L.LNBNN_MODE_BIT(NB))
    try:
        got = L.lnbnn_classify(ix, Q, off, 10, NB, flags=L.LNBNN_TIMING)
        assert L.lnbnn_last_timing(ix)["tile_variant"] == variant
    finally:
        ix.free()
    _, _, D = oracle.knn_class_block(Q, R, labels, classes, 1)
    tot, cls = oracle.nbnn(D, off)
    assert np.array_equal(got[1], tot) and np.array_equal(got[0], cls)


ROW_CASES = [
    # mode, dim, references, queries, k, variant of lists of rows, or None
    (F16, 128, 3200, 900, 1, 6), (F16, 128, 3201, 900, 1, None), (BF16, 128, 6400, 50_000, 1, 6),
    (F16, 128, 4500, 100_000, 1, 2), (F16, 128, 4501, 100_000, 1, None), (F16, 128, 700, 20_000, 5, 2),
    (F16, 128, 700, 19_999, 5, None), (BF16, 128, 1100, 50_000, 10, 2), (F16, 128, 1101, 50_000, 10, None),
    (F16, 128, 1100, 100_000, 15, 2), (F16, 128, 1000, 60_000, 20, None), (F16, 128, 3200, 20_000, 2, 2),
    (I8, 128, 3200, 1000, 1, 11), (I8, 128, 3200, 999, 1, None), (I8, 160, 1100, 100_000, 1, 2),
    (I8, 128, 320, 50_000, 10, 11), (I8, 128, 321, 50_000, 10, None), (I8, 160, 640, 100_000, 5, 2),
    (I8, 128, 320, 100_000, 15, 2), (I8, 160, 320, 60_000, 20, None),
]


@pytest.mark.parametrize("mode,dim,n_refs,n_q,k,variant", ROW_CASES)
def test_lists_of_rows_or_tiles(mode, dim, n_refs, n_q, k, variant):
    R, labels, Q, off = _set(n_refs, n_q, dim)
    tiles = 19 if dim == 160 else 25 if mode == I8 else 26
    ix = L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode))
    try:
        _say(f"small index mode={mode} dim={dim} refs={n_refs} queries={n_q} k={k}")
        got = L.lnbnn_classify(ix, Q, off, k, mode, flags=L.LNBNN_TIMING, want_neighbours=True)
        ran = L.lnbnn_last_timing(ix)["tile_variant"]
        L.lnbnn_set_tuning(ix, mode, k, variant=tiles)
        want = L.lnbnn_classify(ix, Q, off, k, mode, want_neighbours=True)
    finally:
        ix.free()
    assert ran == variant if variant is not None else ran in (19, 25, 26, 28)
    for x, y in zip(want, got):
        assert np.array_equal(x, y)
    _check_head(got, R, labels, Q, k)


@pytest.mark.parametrize("mode,n_refs,k,sizes", [
    (F16, 1000, 10, (33_000, 49_999, 50_000, 65_000, 900, 99_999, 100_000, 131_072)),
    (I8, 300, 10, (33_000, 49_999, 50_000, 65_537, 99_999, 100_000, 131_072)),
    (F16, 3000, 2, (1, 600, 19_999, 20_000, 40_000)),
])
def test_served_batches_of_every_shape(mode, n_refs, k, sizes):
    """The serving slots' buffers hold the lists of whatever shape a batch's size
    picks within its bucket."""
    import time
    R, labels, Q, off = _set(n_refs, max(sizes))
    ix = L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode))
    try:
        L.lnbnn_serve_config(ix, max_batch_desc=1 << 17, max_inflight=1)
        for n in sizes:
            _say(f"served mode={mode} refs={n_refs} k={k} queries={n}")
            t = L.lnbnn_submit(ix, Q[:n], k, mode)
            t0 = time.time()
            while (r := L.lnbnn_poll(ix, t)) is None:
                assert time.time() - t0 < 30
                time.sleep(0.0005)
            want = L.lnbnn_classify(ix, Q[:n], np.array([0, n], np.int64), k, mode)
            assert r[0] == want[0][0] and np.array_equal(r[1], want[1][0])
    finally:
        ix.free()
