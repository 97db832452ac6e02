"""A workspace holds no room for shapes that cannot run."""
import numpy as np
import pytest

import paper_1112_0059_amd as L

pytestmark = pytest.mark.gpu
I8 = L.LNBNN_EXACT_I8


def _index(n, mode=I8, **kw):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    R = torch.randint(0, 256, (n, 128), generator=g, device="cuda", dtype=torch.uint8)
    labels = (torch.arange(n, device="cuda") % 7).to(torch.int32)
    return L.lnbnn_build_index(R, labels, 7, L.LNBNN_MODE_BIT(mode), **kw)


def _free_bytes():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def test_workspace_of_long_lists():
    """INT8 lists of 33 have no shape of 1,024-query blocks: the workspace of a
    small batch holds one list per piece of a 512-query block."""
    ix = _index(1_000_000)
    Q = np.random.default_rng(1).integers(0, 256, size=(900, 128), dtype=np.uint8)
    before = _free_bytes()
    L.lnbnn_classify(ix, Q, np.array([0, 900], np.int64), 32, I8)
    used = before - _free_bytes()
    ix.free()
    # 2 blocks in at most 258 pieces of 512 lists of 33 (key, tile) pairs: 35 MB
    assert used < 52 << 20
