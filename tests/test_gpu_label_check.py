"""Labels that come as device memory are checked on the device: the first one out
of range is named, and nothing is built."""
import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [L.LNBNN_EXACT_I8, L.LNBNN_EXACT_F16, L.LNBNN_NBNN_I8])
@pytest.mark.parametrize("bad", [{}, {0: -1}, {4999: 7}, {1234: 7, 4000: -5}, {2047: 2**31 - 1, 2048: -1}])
def test_device_labels(mode, bad):
    import torch
    R = torch.randint(0, 256, (5000, 128), dtype=torch.uint8, device="cuda")
    labels = (torch.arange(5000, device="cuda") % 7).to(torch.int32)
    for j, v in bad.items():
        labels[j] = v
    if not bad:
        L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode)).free()
        return
    with pytest.raises(L.LnbnnError) as e:
        L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode))
    j = min(bad)
    assert e.value.code == L.LNBNN_EINVAL and f"label[{j}] = {bad[j]} " in str(e.value)
