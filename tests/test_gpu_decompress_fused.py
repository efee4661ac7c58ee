"""Stand-alone decompression in 128-column blocks (outputs that fill more than
half the chip): bitwise the M_hat of the fused step that wrote the factors, with
split products for bf16 M and fp32 products for fp32 M, and the bf16 output is
that M_hat rounded to nearest even.  Widths of whole blocks and not, ranks
padded and not; rows that end inside a tile.
"""

import pytest

from gpu_util import torch_mod
from test_gpu_alignment import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [20, 32, 50, 64, 100, 128])
@pytest.mark.parametrize("shape", [(16500, 392), (33000, 384)])
def test_large_decompress_equals_fused(shape, rank, dtype):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = shape
    M, err, Q = _inputs(m, n, dtype, rank)
    P, Mh = optcc.occ_step(M, err, Q, rank, 1)
    split = optcc.OCC_DEC_SPLIT_BF16 if dtype == "bf16" else 0
    assert torch.equal(optcc.occ_decompress_ex(P, Q, split), Mh)
    out = torch.empty((m, n), device="cuda", dtype=torch.bfloat16)
    optcc.occ_decompress_ex(P, Q, split | optcc.OCC_DEC_OUT_BF16, M_hat=out)
    assert torch.equal(out, Mh.bfloat16())
