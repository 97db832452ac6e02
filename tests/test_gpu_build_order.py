"""An index built from device memory waits for the work of the process's blocking
streams, in which its inputs may still be written."""
import ctypes

import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [L.LNBNN_EXACT_I8, L.LNBNN_EXACT_F16, L.LNBNN_NBNN_I8])
@pytest.mark.parametrize("own_stream", [True, False])
def test_inputs_written_on_a_blocking_stream(mode, own_stream):
    import torch
    n = 50_000
    g = torch.Generator(device="cuda").manual_seed(6)
    R = torch.randint(0, 256, (n, 128), generator=g, device="cuda", dtype=torch.uint8)
    labels = (torch.arange(n, device="cuda") % 7).to(torch.int32)
    Q = (R[:500] ^ 1).contiguous()
    off = np.array([0, 500], np.int64)
    ref = L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode))
    want = L.lnbnn_classify(ref, Q, off, 10, mode)
    torch.cuda.synchronize()
    # the index's own stream is a blocking one
    s = ctypes.c_void_p()
    assert L.load().lnbnn_index_stream(ref.handle, ctypes.byref(s)) == L.LNBNN_OK
    blocking = torch.cuda.ExternalStream(s.value)
    R2, labels2 = torch.zeros_like(R), torch.zeros_like(labels)
    torch.cuda.synchronize()
    with torch.cuda.stream(blocking):
        torch.cuda._sleep(200_000_000)              # about 0.1 s
        R2.copy_(R)
        labels2.copy_(labels)
    side = None if own_stream else torch.cuda.Stream().cuda_stream
    ix = L.lnbnn_build_index(R2, labels2, 7, L.LNBNN_MODE_BIT(mode), stream=side)
    got = L.lnbnn_classify(ix, Q, off, 10, mode)
    torch.cuda.synchronize()
    for x, y in zip(want[:2], got[:2]):
        assert torch.equal(x, y)
    ix.free()
    ref.free()
