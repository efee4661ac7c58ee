"""A warm start Q at any element of a buffer (a view into a flat factor buffer):
bitwise the results of an aligned Q, and nothing written outside Q.  At rank
<= 16 the left product's tiles take such a Q in 4-byte pieces, in the first
round only (the second reads the padded copy); above it the fp32 step copies it
instead of reading it in place.  One batch mixes both kinds.
"""

import pytest

from gpu_util import torch_mod
from test_gpu_alignment import _inputs, _placed, _untouched

pytestmark = pytest.mark.gpu


# whole 32-column steps (LDS tiles) with fewer and more of them than waves and
# stages, and a width without
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [1, 3, 4, 5, 8, 9, 12, 16, 32, 64, 128])
@pytest.mark.parametrize("shape", [(130, 32), (33, 64), (300, 128), (257, 544), (200, 200)])
def test_q_at_any_element(shape, rank, dtype):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = shape
    if rank > min(m, n):
        pytest.skip("rank exceeds the matrix")
    M, err, Q0 = _inputs(m, n, dtype, rank)
    ea, Qa, Ha = err.clone(), Q0.clone(), torch.empty_like(err)
    Pa, _ = optcc.occ_step(M, ea, Qa, rank, 2, M_hat=Ha)
    for off in (1, 2, 3):
        eu, Hu = err.clone(), torch.empty_like(err)
        Qu, qbuf = _placed(Q0, off, rank)
        Pu, _ = optcc.occ_step(M, eu, Qu, rank, 2, M_hat=Hu)
        torch.cuda.synchronize()
        where = f"{shape} r{rank} {dtype} offset {off}"
        assert torch.equal(Pu, Pa) and torch.equal(Qu, Qa), where
        assert torch.equal(eu, ea) and torch.equal(Hu, Ha), where
        assert _untouched(Qu, qbuf), where


@pytest.mark.parametrize("rank", [3, 16, 64])
def test_batch_of_aligned_and_unaligned_q(rank):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    shapes = [(300, 128), (257, 544), (130, 96)]
    outs = []
    for off in (0, 1):
        items = []
        for j, (m, n) in enumerate(shapes):
            M, err, Q0 = _inputs(m, n, "f32", rank)
            Q, _ = _placed(Q0, off if j == 1 else 0, rank)
            items.append((M, err, Q, torch.empty((m, rank), device="cuda"), torch.empty_like(err)))
        optcc.occ_step_batched(items, rank, 2)
        torch.cuda.synchronize()
        outs.append([t for it in items for t in it])
    assert all(torch.equal(a, b) for a, b in zip(*outs))
