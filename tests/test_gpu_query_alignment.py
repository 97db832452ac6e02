"""Device queries at any address: a contiguous view may start at any byte of its
storage, and the results are those of an aligned copy."""
import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu

I8, F16, BF16, NB, FP8 = (L.LNBNN_EXACT_I8, L.LNBNN_EXACT_F16, L.LNBNN_EXACT_BF16, L.LNBNN_NBNN_I8,
                          L.LNBNN_FP8_RERANK)


@pytest.mark.parametrize("mode,dim", [(I8, 128), (I8, 160), (F16, 128), (BF16, 128), (NB, 128), (FP8, 128)])
@pytest.mark.parametrize("shift", [1, 2, 3, 4, 8])
def test_shifted_queries(mode, dim, shift):
    import torch
    fl = mode == FP8
    if fl and shift % 4:
        pytest.skip("floats stand on 4-byte addresses")
    g = torch.Generator(device="cuda").manual_seed(17)
    R = torch.randint(0, 256, (6007, dim), generator=g, device="cuda").to(torch.float32 if fl else torch.uint8)
    labels = (torch.arange(6007, device="cuda") % 7).to(torch.int32)
    Q = torch.randint(0, 256, (333, dim), generator=g, device="cuda").to(R.dtype)
    off = np.array([0, 100, 333], np.int64)
    step = shift // 4 if fl else shift
    buf = torch.full((Q.numel() + step,), 77, dtype=Q.dtype, device="cuda")
    view = buf[step:].view(Q.shape)
    view.copy_(Q)
    assert view.data_ptr() % 16 == shift
    ix = L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode))
    nbr = mode != NB
    try:
        for flags in (0, L.LNBNN_PER_IMAGE_LAUNCH):
            want = L.lnbnn_classify(ix, Q, off, 10, mode, flags=flags, want_neighbours=nbr)
            got = L.lnbnn_classify(ix, view, off, 10, mode, flags=flags, want_neighbours=nbr)
            for x, y in zip(want, got):
                assert x is None or torch.equal(x, y)
        out = {"class": torch.empty_like(want[0]), "totals": torch.empty_like(want[1])}
        L.lnbnn_classify_noalloc(ix, view, off, 10, mode, out)
        assert torch.equal(out["class"], want[0]) and torch.equal(out["totals"], want[1])
    finally:
        torch.cuda.synchronize()
        ix.free()
