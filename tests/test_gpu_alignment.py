"""Rows at element alignment: any base offset and any leading dimension gives
bitwise the outputs of the same step on 16-byte aligned rows, and writes
nothing outside the m x n elements of err and M_hat.

The vector loads and stores of both forms carry the same values into the same
products, so the comparison is exact; the aligned form is checked against the
float64 oracle in test_gpu_parity.py.
"""

import pytest

from gpu_util import torch_mod

pytestmark = pytest.mark.gpu

SENTINEL = 4096.0   # exact in bf16 too


def _placed(x, offset: int, ld: int):
    """x (m x n) at element `offset` of a sentinel-filled buffer, pitch ld: (view, buffer)."""
    torch = torch_mod()
    m, n = x.shape
    buf = torch.full((offset + m * ld + 64,), SENTINEL, dtype=x.dtype, device="cuda")
    view = buf.as_strided((m, n), (ld, 1), offset)
    view.copy_(x)
    return view, buf


def _untouched(view, buf) -> bool:
    torch = torch_mod()
    mask = torch.ones_like(buf, dtype=torch.bool)
    mask.as_strided(view.shape, view.stride(), view.storage_offset())[:] = False
    return bool((buf[mask] == SENTINEL).all())


def _inputs(m, n, dtype, rank):
    torch = torch_mod()
    g = torch.Generator(device="cuda")
    g.manual_seed(m * 131 + n * 7 + rank)
    M = torch.randn((m, n), generator=g, device="cuda")
    if dtype == "bf16":
        M = M.bfloat16()
    err = 0.1 * torch.randn((m, n), generator=g, device="cuda")
    return M, err, torch.randn((n, rank), generator=g, device="cuda")


def _step(M, err, Q, rank, iters, M_hat):
    from paper_2301_09830_amd import optcc
    Q = Q.clone()
    P, _ = optcc.occ_step(M, err, Q, rank, iters, M_hat=M_hat)
    torch_mod().cuda.synchronize()
    return P, Q


# (m, n): one row tile and less, remainders of the 16-, 32-, 64- and 128-wide
# tiles, fewer columns than one vector, whole tiles at an odd pitch
SHAPES = [(16, 16), (33, 31), (130, 97), (70, 257), (257, 128), (300, 395)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [3, 8, 16, 17, 48, 128])
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_at_element_alignment(shape, rank, dtype):
    torch = torch_mod()
    m, n = shape
    if rank > min(m, n):
        pytest.skip("rank exceeds the matrix")
    M, err, Q = _inputs(m, n, dtype, rank)
    ld = (n + 7) // 8 * 8                     # aligned rows
    Ma, _ = _placed(M, 0, ld)
    ea, ebuf = _placed(err, 0, ld)
    ha, _ = _placed(torch.zeros_like(err), 0, ld)
    Pa, Qa = _step(Ma, ea, Q, rank, 2, ha)
    for off in (1, 2, 3, 5):
        for pad in (0, 1, 3):
            Mu, _ = _placed(M, off, n + pad)
            eu, ebuf = _placed(err, off, n + pad)
            hu, hbuf = _placed(torch.zeros_like(err), off, n + pad)
            Pu, Qu = _step(Mu, eu, Q, rank, 2, hu)
            where = f"{shape} r{rank} {dtype} offset {off} pad {pad}"
            assert torch.equal(Pu, Pa) and torch.equal(Qu, Qa), where
            assert torch.equal(eu, ea) and torch.equal(hu, ha), where
            assert _untouched(eu, ebuf) and _untouched(hu, hbuf), where
