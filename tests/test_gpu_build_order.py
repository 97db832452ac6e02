"""An index built from device memory waits for the work of the process's blocking
streams, in which its inputs may still be written, and names the first label out of
range, whether few labels are read back or many are checked on the device."""
import ctypes

import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [L.LNBNN_EXACT_I8, L.LNBNN_EXACT_F16, L.LNBNN_NBNN_I8])
@pytest.mark.parametrize("own_stream", [True, False])
@pytest.mark.parametrize("n", [50_000, 8_000])
def test_inputs_written_on_a_blocking_stream(mode, own_stream, n):
    import torch
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


@pytest.mark.parametrize("mode", [L.LNBNN_EXACT_I8, L.LNBNN_NBNN_I8])
@pytest.mark.parametrize("n", [8192, 8193])
@pytest.mark.parametrize("bad", [{}, {0: -1}, {8191: 7}, {1234: 7, 8000: -5}])
def test_first_bad_label(mode, n, bad):
    import torch
    R = torch.randint(0, 256, (n, 128), dtype=torch.uint8, device="cuda")
    labels = (torch.arange(n, device="cuda") % 7).to(torch.int32)
    for j, v in bad.items():
        labels[j] = v
    if not bad:
        L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode)).free()
        return
    with pytest.raises(L.LnbnnError) as e:
        L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode))
    j = min(bad)
    assert e.value.code == L.LNBNN_EINVAL and f"label[{j}] = {bad[j]} " in str(e.value)
