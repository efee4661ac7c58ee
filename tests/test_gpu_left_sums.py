"""The left product of one fp32 matrix above rank 16, where the plan gives a
block more columns than it sums at once: P_hat, Q, M_hat and err against
float64, at the error that sums of that length have.

An fp32 sum of k products in sequence is off by about sqrt(k) eps of its terms,
so a sum of twice the columns adds up to 40 % to the left product's part of the
error.  The bounds are 10 % above the errors measured with sums of the columns
of the splits before they were merged (3.8e-7, 6.0e-7, 5.4e-7, 4.2e-7, 5.6e-7);
in one sum over a block's columns the first two were 4.4e-7 and 8.0e-7.
"""

import pytest

from gpu_util import torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,rank,bound", [((5003, 2047), 48, 4.2e-7), ((3722, 8120), 41, 6.6e-7),
                                              ((3467, 4736), 32, 5.9e-7), ((5003, 2047), 128, 4.6e-7),
                                              ((3467, 4736), 100, 6.2e-7)])
def test_error_of_merged_splits(shape, rank, bound):
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
    assert rel <= bound
    # the compress-only call runs the same sums
    Mc = 1e-3 * torch.randn((m, n), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    ec = 0.5 * Mc.flip(0)
    Qc, Qf = Q0.float(), Q0.float()
    Pc = optcc.occ_compress(Mc, ec, Qc, rank, 1)
    Pf, _ = optcc.occ_step(Mc, ec, Qf, rank, 1)
    assert torch.equal(Pc, Pf) and torch.equal(Qc, Qf)
