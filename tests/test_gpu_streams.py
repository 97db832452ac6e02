"""Calls of two indexes in flight at once: each index runs on its own stream, so
a dropped output's memory must not be given to another index's call while the
first still writes it."""
import numpy as np
import pytest

import oracle
import paper_1112_0059_amd as L
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [L.LNBNN_EXACT_I8, L.LNBNN_EXACT_F16])
def test_dropped_outputs_of_two_indexes(mode):
    import torch
    sets = []
    for seed in (1, 2):
        cfg = synth.scaled(synth.CONFIGS["T"], n_img=1, index_seed=100 + seed, query_seed=200 + seed)
        R, labels = synth.gen_index(cfg)
        Q, off, _ = synth.gen_queries(cfg)
        ix = L.lnbnn_build_index(R, labels, cfg.n_classes, L.LNBNN_MODE_BIT(mode))
        sets.append((ix, torch.from_numpy(Q).cuda(), off, oracle.classify(Q, R, labels, cfg.n_classes, off, 10)))
    try:
        for rep in range(60):
            got = []
            for ix, dq, off, want in (sets[0], sets[1], sets[0]):
                out = L.lnbnn_classify(ix, dq, off, 10, mode, want_neighbours=True)   # the ones before are dropped
            ix, dq, off, (wt, wc, wi, wd) = sets[0]
            cls, tot, ni, nd = (x.cpu().numpy() for x in out)
            assert np.array_equal(ni, wi) and np.array_equal(nd.astype(np.int64), wd), rep
            assert np.array_equal(tot, wt) and np.array_equal(cls, wc), rep
            # outputs that outlive their index
            del out
    finally:
        for s in sets:
            s[0].free()
