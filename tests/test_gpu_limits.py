"""Rows and columns up to the largest accepted count, 2^31 - 1: the calls that
take such a matrix in the memory of one GPU (the decompression at the smallest
rank and the error update).  Row and column numbers one tile, group or chunk
past the last one no longer fit 32 signed bits there.

Inputs are small whole numbers, so every product and sum is exact and compared
for equality over the whole output; elements after the output stay untouched.
"""

import pytest

from gpu_util import torch_mod

pytestmark = pytest.mark.gpu

MOST = 2 ** 31 - 1
GUARD = 64
SENTINEL = 77.0


def _numbers(count, mod, dtype):
    """0, 1, .. mod - 1, 0, .. as `dtype`, with a guarded end: (values, buffer)."""
    torch = torch_mod()
    buf = torch.empty(count + GUARD, dtype=dtype, device="cuda")
    for lo in range(0, count, 1 << 28):
        hi = min(count, lo + (1 << 28))
        buf[lo:hi] = torch.arange(lo, hi, device="cuda").remainder_(mod).to(dtype)
    buf[count:] = SENTINEL
    return buf[:count], buf


def _same(got, want_of, count):
    for lo in range(0, count, 1 << 28):
        hi = min(count, lo + (1 << 28))
        if not bool((got[lo:hi] == want_of(lo, hi)).all()):
            return False
    return True


@pytest.mark.parametrize("bf16", [False, True])
# (wide: 2^24 - 1 column tiles of 128, the most blocks of 256 threads that a launch takes)
@pytest.mark.parametrize("count,tall", [(MOST, True), (MOST - 64, True), (MOST - 127, False)])
def test_decompress_most_rows_or_columns(count, tall, bf16):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    dt = torch.bfloat16 if bf16 else torch.float32
    long, _ = _numbers(count, 61, torch.float32)
    one = torch.full((1, 1), 3.0, device="cuda")
    out = torch.full((count + GUARD,), SENTINEL, dtype=dt, device="cuda")
    m, n = (count, 1) if tall else (1, count)
    P, Q = (long.view(m, 1), one) if tall else (one, long.view(n, 1))
    optcc.occ_decompress_ex(P, Q, optcc.OCC_DEC_OUT_BF16 if bf16 else 0,
                            M_hat=out[:count].view(m, n))
    torch.cuda.synchronize()
    assert _same(out, lambda lo, hi: (3.0 * long[lo:hi]).to(dt), count)
    assert bool((out[count:] == SENTINEL).all())


@pytest.mark.parametrize("tall", [True, False])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_err_update_most_rows_or_columns(dtype, tall):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = (MOST, 1) if tall else (1, MOST)
    M, _ = _numbers(MOST, 61, torch.bfloat16 if dtype == "bf16" else torch.float32)
    mh, _ = _numbers(MOST, 59, torch.float32)
    err, buf = _numbers(MOST, 53, torch.float32)
    optcc.occ_err_update(M.view(m, n), err.view(m, n), mh.view(m, n), err_new=err.view(m, n))
    torch.cuda.synchronize()

    def want(lo, hi):
        e = torch.arange(lo, hi, device="cuda").remainder_(53).float()
        return M[lo:hi].float() + e - mh[lo:hi]

    assert _same(err, want, MOST)
    assert bool((buf[MOST:] == SENTINEL).all())
