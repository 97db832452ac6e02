"""An index's own stream outlives the index: outputs that torch holds for that stream
stay whole after the index is freed and another one runs."""
import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu


def test_outputs_that_outlive_their_index():
    import torch
    g = torch.Generator(device="cuda").manual_seed(2)
    sets = []
    for _ in range(2):
        R = torch.randint(0, 256, (200_000, 128), generator=g, device="cuda", dtype=torch.uint8)
        labels = (torch.arange(R.shape[0], device="cuda") % 9).to(torch.int32)
        sets.append((R, labels, R[:4000] ^ 3))
    off = np.array([0, 1000, 4000], np.int64)

    def run(s):
        ix = L.lnbnn_build_index(s[0], s[1], 9, L.LNBNN_MODE_BIT(L.LNBNN_EXACT_I8))
        return ix, L.lnbnn_classify(ix, s[2], off, 10, L.LNBNN_EXACT_I8, want_neighbours=True)

    want = []
    for s in sets:
        ix, out = run(s)
        torch.cuda.synchronize()
        want.append([x.clone() for x in out])
        ix.free()
    for rep in range(20):
        ix, first = run(sets[0])
        ix.free()                                   # the outputs are still held for its stream
        ix, second = run(sets[1])                   # on the same stream, in the same buffers
        keep = [x.clone() for x in first]
        del first                                   # their memory waits for that stream,
        junk = [torch.full((4000, 11), -1, dtype=torch.int32, device="cuda") for _ in range(4)]   # and is reused
        torch.cuda.synchronize()
        for x, y in zip(want[0], keep):
            assert torch.equal(x, y), rep
        for x, y in zip(want[1], second):
            assert torch.equal(x, y), rep
        assert all(int(j.max()) == -1 for j in junk)
        ix.free()
