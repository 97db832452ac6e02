"""Device memory around an index's life: buffers kept after an index is freed are
neither hidden from the next index's budget nor lost to the rest of the process,
and a kept buffer is never given out where a smaller one was asked for."""
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


def test_kept_buffers_can_be_given_back():
    _index(5000).free()                      # the library's first use, once per process
    L.lnbnn_trim()
    before = _free_bytes()
    _index(4_000_000).free()
    kept = before - _free_bytes()
    L.lnbnn_trim()
    after = _free_bytes()
    assert kept > 400 << 20                  # the rows alone are 512 MB
    assert before - after < 64 << 20
    L.lnbnn_trim()                           # nothing kept: nothing happens


def test_kept_buffers_count_as_free_for_the_budget():
    _index(5000).free()
    L.lnbnn_trim()
    budgets = []
    for _ in range(2):                       # nothing kept, then a large index's buffers
        _free_bytes()                        # and torch's own cache is empty
        ix = _index(5000)
        budgets.append(L.lnbnn_serve_info(ix)["hbm_budget"])
        ix.free()
        _index(6_000_000).free()
    L.lnbnn_trim()
    assert abs(budgets[0] - budgets[1]) < 32 << 20


def test_buffers_are_no_larger_than_asked_for():
    """An index rebuilt a little smaller holds its own size: the serving slots'
    accounting counts what was asked for."""
    _index(5000).free()
    L.lnbnn_trim()
    before = _free_bytes()
    _index(4_000_000).free()
    ix = _index(3_400_000)
    L.lnbnn_trim()                           # what is kept beside it
    held = before - _free_bytes()
    assert held < L.lnbnn_index_info(ix)["device_bytes"] + (48 << 20)
    ix.free()
    L.lnbnn_trim()
