"""The left product of one fp32 matrix above rank 16, where the plan gives a
block more columns than it sums at once: P_hat, Q, M_hat and err against
float64, at the error that sums of that length have.

The bound is the random-walk error of fp32 sums: k products summed in sequence
are off by about sqrt(k / 3) eps / 2 of their root mean square each; with at
most 256 columns a sum, 16 partial sums of it and the same again for the right
product, M_hat stays below 6e-7 on noise (measured 4.0e-7 to 4.5e-7 in sums of
256 columns; in one sum over a block's columns, 4.4e-7 to 8.0e-7).
"""

import pytest

from gpu_util import torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,rank", [((5003, 2047), 48), ((3722, 8120), 41), ((3467, 4736), 32),
                                        ((5003, 2047), 128), ((3467, 4736), 100)])
def test_error_of_merged_splits(shape, rank):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    m, n = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n + rank)
    M = 1e-3 * torch.randn((m, n), generator=g, device="cuda")
    err = 1e-3 * torch.randn((m, n), generator=g, device="cuda")
    Q = torch.randn((n, rank), generator=g, device="cuda")
    A, Q0 = M.double() + err.double(), Q.double()
    P, Mh = optcc.occ_step(M, err, Q, rank, 1)
    p = torch.linalg.qr(A @ Q0)[0]
    ref = p @ (A.T @ p).T
    rel = ((Mh.double() - ref).norm() / ref.norm()).item()
    print(f"[sums] {m}x{n} r{rank}: M_hat {rel:.3e}", flush=True)
    assert rel <= 6e-7
    # the compress-only call runs the same sums
    Mc = 1e-3 * torch.randn((m, n), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    ec = 0.5 * Mc.flip(0)
    Qc, Qf = Q0.float(), Q0.float()
    Pc = optcc.occ_compress(Mc, ec, Qc, rank, 1)
    Pf, _ = optcc.occ_step(Mc, ec, Qf, rank, 1)
    assert torch.equal(Pc, Pf) and torch.equal(Qc, Qf)
