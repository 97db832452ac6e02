"""Float references with a NaN or an infinity are neighbours of nothing, and
the references packed beside them are found as if those rows were far away."""
import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu
FP8, FP8_2K = L.LNBNN_FP8_RERANK, L.LNBNN_FP8_RERANK_2K


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("mode,k,variant", [(FP8, 1, -1), (FP8, 10, -1), (FP8, 16, -1), (FP8, 10, 0), (FP8, 10, 27),
                                            (FP8_2K, 10, -1), (FP8_2K, 3, -1)])
def test_rows_beside_a_nonfinite_one(mode, k, variant, value):
    rng = np.random.default_rng(23)
    R = np.maximum(rng.standard_normal((9001, 128)), 0).astype(np.float32)
    labels = rng.integers(0, 9, size=R.shape[0]).astype(np.int32)
    Q = np.maximum(R[rng.integers(0, R.shape[0], size=700)] + 0.1 * rng.standard_normal((700, 128)), 0)
    Q = Q.astype(np.float32)
    off = np.array([0, 300, 700], np.int64)
    bad = np.r_[5:R.shape[0]:64, 9000]       # every other tile, and the last row
    far, odd = R.copy(), R.copy()
    far[bad] = 100.0
    odd[bad, rng.integers(0, 128, size=bad.size)] = value
    odd[bad[0]] = value                      # a whole row
    res = []
    for refs in (far, odd):
        ix = L.lnbnn_build_index(refs, labels, 9, L.LNBNN_MODE_BIT(mode))
        try:
            L.lnbnn_set_tuning(ix, mode, k, variant=variant)
            res.append(L.lnbnn_classify(ix, Q, off, k, mode, want_neighbours=True))
        finally:
            ix.free()
    assert not np.isin(res[0][2], bad).any()
    for x, y in zip(*res):
        assert np.array_equal(x, y)
