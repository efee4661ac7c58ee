"""Decompression above rank 16 at the ends of the factors: at ranks that are not
padded the last rows of P and Q are read in whole vectors taken from inside the
arrays.  Elements after each factor are NaN (a value taken from there shows in
the output), the last rows differ from all others, and the products are whole
numbers small enough to be exact in fp32 and in split bf16, so the outputs are
compared for equality.
"""

import pytest

from gpu_util import torch_mod

pytestmark = pytest.mark.gpu


# up to 3 elements of a vector past the end (rank mod 4), padded ranks 32 to
# 128, one row tile and less, whole tiles and one row more, 64- and 128-column
# blocks
@pytest.mark.parametrize("rank", [17, 18, 19, 20, 31, 33, 47, 61, 65, 100, 127])
@pytest.mark.parametrize("shape", [(127, 127), (128, 128), (129, 191), (300, 129), (16500, 392)])
def test_factor_ends(shape, rank):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = shape
    if rank > min(m, n):
        pytest.skip("rank exceeds the matrix")
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n + rank)

    def factor(rows):
        buf = torch.full((rows * rank + 64,), float("nan"), device="cuda")
        f = buf[:rows * rank].view(rows, rank)
        f.copy_(torch.randint(-3, 4, (rows, rank), generator=g, device="cuda"))
        f[-1] = torch.arange(rank, device="cuda") % 7 + 1
        return f

    P, Q = factor(m), factor(n)
    want = (P.double() @ Q.double().T).float()
    for split in (0, optcc.OCC_DEC_SPLIT_BF16):
        out = optcc.occ_decompress_ex(P, Q, split)
        assert torch.equal(out, want), f"{shape} r{rank} split {split}"
