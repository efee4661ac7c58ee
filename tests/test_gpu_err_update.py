"""Stand-alone error update over the edges of its four-column chunks: any row
alignment, rows that end inside a chunk, in place and out of place, without an
error buffer.  The kernel adds and subtracts in the order of the formula, so
the result is bitwise that of the same fp32 operations in torch.
"""

import pytest

from gpu_util import torch_mod
from test_gpu_alignment import _placed, _untouched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 1), (3, 4), (5, 7), (64, 130), (1030, 33), (700, 1024)])
def test_err_update_edges(shape, dtype):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(m * 31 + n)
    M = torch.randn((m, n), generator=g, device="cuda")
    M = M.bfloat16() if dtype == "bf16" else M
    err = torch.randn((m, n), generator=g, device="cuda")
    mh = torch.randn((m, n), generator=g, device="cuda")
    for off, pad in ((0, 0), (1, 0), (2, 3), (16, 16)):
        Mv, _ = _placed(M, off, n + pad)
        hv, _ = _placed(mh, off, n + pad)
        ev, ebuf = _placed(err, off, n + pad)
        want = (M.float() + err) - mh
        ov, obuf = _placed(torch.zeros_like(err), off, n + pad)
        optcc.occ_err_update(Mv, ev, hv, err_new=ov)
        assert torch.equal(ov, want) and _untouched(ov, obuf)
        optcc.occ_err_update(Mv, ev, hv, err_new=ev)
        assert torch.equal(ev, want) and _untouched(ev, ebuf)
        optcc.occ_err_update(Mv, None, hv, err_new=ov)
        assert torch.equal(ov, M.float() - mh) and _untouched(ov, obuf)
