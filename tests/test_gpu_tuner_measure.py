"""The autotuner ranks settings by the time of the whole search: shared lists
leave part of it (the rows of the best tiles) to a kernel after the distance
kernel, per-row lists do not."""
import re

import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,k,n_refs,n_q", [(L.LNBNN_EXACT_F16, 32, 1000, 60_000), (L.LNBNN_EXACT_I8, 10, 40_000, 20_000),
                                               (L.LNBNN_FP8_RERANK, 5, 20_000, 20_000)])
def test_ranked_by_the_whole_call(mode, k, n_refs, n_q, capfd, monkeypatch):
    import torch
    monkeypatch.setenv("LNBNN_LOG", "1")
    monkeypatch.delenv("LNBNN_TUNE_CACHE", raising=False)
    fl = mode == L.LNBNN_FP8_RERANK
    g = torch.Generator(device="cuda").manual_seed(9)
    R = torch.randint(0, 256, (n_refs, 128), generator=g, device="cuda").to(torch.float32 if fl else torch.uint8)
    labels = (torch.arange(n_refs, device="cuda") % 7).to(torch.int32)
    Q = torch.randint(0, 256, (n_q, 128), generator=g, device="cuda").to(R.dtype)
    off = np.array([0, n_q // 3, n_q], np.int64)
    ix = L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode))
    try:
        best = L.lnbnn_variant_name(L.lnbnn_autotune(ix, Q, off, k, mode))
    finally:
        ix.free()
    log = capfd.readouterr().err
    runs = re.findall(r"tuner: mode \d+, k \d+: (\S+), chunk (\d+): ([\d.]+) ms, distance kernel ([\d.]+) ms", log)
    assert len(runs) >= 3, log
    times = {(n, int(c)): float(t) for n, c, t, _ in runs}
    assert all(float(t) > float(d) > 0 for _, _, t, d in runs)
    chosen = re.search(r"-> (\S+), chunk (\d+) \(", log)
    assert chosen.group(1) == best
    # the printed times are rounded to 10 us
    assert times[best, int(chosen.group(2))] <= min(times.values()) + 0.011
