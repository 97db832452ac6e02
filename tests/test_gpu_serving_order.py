"""A batch is published when its own work is done, not when the batch after it
is: the short kernels that finish a batch must not wait for the next batch's
sweep of the index, which leaves them no room on the compute units."""
import sys
import time

import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu

N_Q = 32768


def _wait(ix, tickets):
    out, t0 = [], time.time()
    for t in tickets:
        while (r := L.lnbnn_poll(ix, t)) is None:
            assert time.time() - t0 < 60
            time.sleep(0.0005)
        out.append(r)
    return out


@pytest.mark.parametrize("mode,k,dim,n_refs", [
    (L.LNBNN_EXACT_I8, 10, 128, 3_000_000),
    (L.LNBNN_EXACT_I8, 20, 128, 3_000_000),
    (L.LNBNN_EXACT_I8, 10, 160, 2_000_000),
    (L.LNBNN_EXACT_F16, 10, 128, 1_500_000),
    (L.LNBNN_NBNN_I8, 10, 128, 3_000_000),
    (L.LNBNN_FP8_RERANK, 5, 128, 2_000_000),
    (L.LNBNN_FP8_RERANK, 10, 128, 2_000_000),
    (L.LNBNN_FP8_RERANK_2K, 10, 128, 2_000_000),
])
def test_batches_finish_one_after_the_other(mode, k, dim, n_refs):
    import torch
    fl = mode in (L.LNBNN_FP8_RERANK, L.LNBNN_FP8_RERANK_2K)
    g = torch.Generator(device="cuda").manual_seed(3)
    if fl:
        R = torch.rand(n_refs, dim, generator=g, device="cuda")
        Q = np.random.default_rng(4).random((N_Q, dim), dtype=np.float32)
    else:
        R = torch.randint(0, 256, (n_refs, dim), generator=g, device="cuda", dtype=torch.uint8)
        Q = np.random.default_rng(4).integers(0, 256, size=(N_Q, dim), dtype=np.uint8)
    labels = (torch.arange(n_refs, device="cuda") % 16).to(torch.int32)
    ix = L.lnbnn_build_index(R, labels, 16, L.LNBNN_MODE_BIT(mode))
    del R, labels
    try:
        L.lnbnn_serve_config(ix, max_batch_desc=N_Q, max_inflight=2)
        _wait(ix, [L.lnbnn_submit(ix, Q, k, mode) for _ in range(4)])       # captures, first passes
        alone = min(st["t_done_ns"] - st["t_start_ns"] for _, _, st in
                    (_wait(ix, [L.lnbnn_submit(ix, Q, k, mode)])[0] for _ in range(3)))
        res = _wait(ix, [L.lnbnn_submit(ix, Q, k, mode) for _ in range(6)])
        done = np.array([st["t_done_ns"] for _, _, st in res])
        gaps = np.diff(done) / alone
        print(f"mode {mode} k {k} dim {dim}: alone {alone / 1e6:.2f} ms, gaps between batches / alone {np.round(gaps, 2)}",
              flush=True)
        sys.stdout.flush()
        assert gaps.min() > 0.5
        for c, tot, _ in res:
            assert c == res[0][0] and np.array_equal(tot, res[0][1])
    finally:
        ix.free()
