"""Stand-alone decompression above rank 16 at the edges of its tiles: the
64- and 128-column blocks (the last shape's blocks fill more
than half the chip), 32-row wave tiles, output pieces of 4 or 8 elements, ranks
that are not padded, factors and outputs at any alignment.

Against float64: an fp32 product of length r with unit-size terms is off by at
most about r eps of the sum of |terms|, a split bf16 product by 2^-16 of it; a
bf16 output adds 2^-9 of its value.  Bitwise equality with the fused step's
M_hat is checked in test_gpu_properties.py (64-column blocks) and
test_gpu_decompress_fused.py (128-column blocks).
"""

import pytest

from gpu_util import torch_mod
from test_gpu_alignment import _placed, _untouched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [17, 32, 50, 64, 100, 128])
@pytest.mark.parametrize("shape", [(128, 128), (129, 131), (257, 160), (160, 1027), (2050, 392),
                                   (16500, 392)])
def test_decompress_edges(shape, rank):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(m * 17 + n * 3 + rank)
    P = torch.randn((m, rank), generator=g, device="cuda")
    Q = torch.randn((n, rank), generator=g, device="cuda")
    want = P.double() @ Q.double().T
    size = P.double().abs() @ Q.double().abs().T      # sum of |terms| of each element
    for split in (0, optcc.OCC_DEC_SPLIT_BF16):
        for out_bf16 in (0, optcc.OCC_DEC_OUT_BF16):
            dt = torch.bfloat16 if out_bf16 else torch.float32
            for off, pad in ((0, 0), (0, 64), (1, 1), (3, 8)):
                Pv = torch.empty(m * rank + off, device="cuda")[off:].view(m, rank).copy_(P)
                out, buf = _placed(torch.zeros((m, n), device="cuda", dtype=dt), off, n + pad)
                optcc.occ_decompress_ex(Pv, Q, split | out_bf16, M_hat=out)
                bound = size * (2.0 ** -15 if split else rank * 2.0 ** -23)
                if out_bf16:
                    bound = bound + want.abs() * 2.0 ** -8
                where = f"{shape} r{rank} split {split} bf16 {out_bf16} offset {off} pad {pad}"
                assert bool(((out.double() - want).abs() <= bound).all()), where
                assert _untouched(out, buf), where
