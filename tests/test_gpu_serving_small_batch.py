"""A served batch of a few query blocks is cut over the whole GPU like the same
batch classified directly, although a slot holds fewer lists per query."""
import time

import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,n_q", [(L.LNBNN_EXACT_I8, 300), (L.LNBNN_EXACT_I8, 1500), (L.LNBNN_EXACT_F16, 700),
                                      (L.LNBNN_FP8_RERANK, 700)])
def test_small_request_on_a_large_index(mode, n_q):
    import torch
    g = torch.Generator(device="cuda").manual_seed(1)
    fl = mode == L.LNBNN_FP8_RERANK
    n = 4_000_000
    R = torch.rand(n, 128, generator=g, device="cuda") if fl else torch.randint(0, 256, (n, 128), generator=g, device="cuda", dtype=torch.uint8)
    labels = (torch.arange(n, device="cuda") % 16).to(torch.int32)
    ix = L.lnbnn_build_index(R, labels, 16, L.LNBNN_MODE_BIT(mode))
    Q = R[:n_q].cpu().numpy()
    del R, labels
    try:
        off = np.array([0, n_q], np.int64)
        direct = 1e9
        for _ in range(3):
            want = L.lnbnn_classify(ix, Q, off, 10, mode, flags=L.LNBNN_TIMING)
            direct = min(direct, L.lnbnn_last_timing(ix)["total_ms"])
        served = 1e9
        for _ in range(5):
            t = L.lnbnn_submit(ix, Q, 10, mode)
            while (r := L.lnbnn_poll(ix, t)) is None:
                time.sleep(0.0005)
            served = min(served, (r[2]["t_done_ns"] - r[2]["t_start_ns"]) / 1e6)
            assert r[0] == want[0][0] and np.array_equal(r[1], want[1][0])
        print(f"mode {mode}, {n_q} descriptors: direct {direct:.2f} ms, served {served:.2f} ms", flush=True)
        # one to three blocks in 64 slices each fill a quarter of the GPU or more
        assert served < 5 * direct + 1.0
    finally:
        ix.free()
