"""Compress-only calls above rank 16 read M and err_prev again in the right
product, through LDS tiles of both.  P_hat and Q are bitwise those of the
fused step, which reads the stored A = M + err_prev instead: same values, same
products, same order.  Sizes at the edges of the column tiles (128 to 512
columns a block) and of the 8- and 16-row groups, widths with whole 32-column
steps (16-byte pieces) and without, aligned and unaligned rows.
"""

import pytest

from gpu_util import torch_mod
from test_gpu_alignment import _inputs, _placed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [17, 32, 64, 100, 128])
@pytest.mark.parametrize("shape", [(128, 128), (129, 160), (263, 544), (1000, 288), (391, 331)])
def test_compress_equals_fused(shape, rank, dtype):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = shape
    M, err, Q0 = _inputs(m, n, dtype, rank)
    for off, ld in ((0, (n + 7) // 8 * 8), (1, n), (8, n + 3)):
        Mv, _ = _placed(M, off, ld)
        ev, _ = _placed(err, off, ld)
        Qc, Qf = Q0.clone(), Q0.clone()
        Pc = optcc.occ_compress(Mv, ev, Qc, rank, 2)
        Pf, _ = optcc.occ_step(Mv, ev, Qf, rank, 2, write_mhat=False)
        torch.cuda.synchronize()
        where = f"{shape} r{rank} {dtype} offset {off} ld {ld}"
        assert torch.equal(Pc, Pf) and torch.equal(Qc, Qf), where
