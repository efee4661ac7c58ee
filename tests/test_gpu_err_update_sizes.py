"""Stand-alone error update on both sides of the size where a thread takes two
chunks of four columns instead of one (2^19 chunks), for rows with and without
a short last chunk and narrower than a chunk, whole rounds of blocks and a
piece of one.  Bitwise the same fp32 operations in torch, in place.
"""

import pytest

from gpu_util import torch_mod
from test_gpu_alignment import _placed, _untouched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(9, 2), (1000, 3), (2048, 1024), (2049, 1024), (1394, 1501),
                                   (1395, 1501), (1400, 1502), (1399, 1503), (600000, 3)])
def test_err_update_sizes(shape, dtype):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    M = torch.randn((m, n), generator=g, device="cuda")
    M = M.bfloat16() if dtype == "bf16" else M
    err = torch.randn((m, n), generator=g, device="cuda")
    mh = torch.randn((m, n), generator=g, device="cuda")
    want = (M.float() + err) - mh
    for off, pad in ((0, 0), (3, 1)):
        Mv, _ = _placed(M, off, n + pad)
        hv, _ = _placed(mh, off, n + pad)
        ev, buf = _placed(err, off, n + pad)
        optcc.occ_err_update(Mv, ev, hv, err_new=ev)
        torch.cuda.synchronize()
        assert torch.equal(ev, want) and _untouched(ev, buf), f"{shape} {dtype} offset {off}"
