"""Second CholeskyQR pass above rank 16, at the row counts where the kernel
that forms its Gram changes: up to 128 rows per Gram block the P_hat kernel
does it beside its own rows (400, 5000 rows), above that (20000 rows) and at
padded rank 128 a kernel of its own; one batch holds both kinds.  Geometric
spectra as in test_ill_conditioned_iterates_second_pass, so the first pass
alone would leave P_hat short of orthonormal.
"""

import numpy as np
import pytest

from gpu_util import assert_parity, run_workload
from workloads import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,ratio", [(32, 1.1), (64, 1.05), (128, 1.025)])
@pytest.mark.parametrize("shapes", [((5000, 160),), ((20000, 160),), ((20000, 160), (400, 300))])
def test_second_pass_gram_kernels(shapes, rank, ratio):
    w = Workload(96, "geom", shapes, "f32", rank, 2, 1, "geom", signal_rank=rank + 8, noise=ratio)
    orth = []

    def on_step(s, j, out, M):
        P = out["P"].astype(np.float64)
        orth.append(np.abs(P.T @ P - np.eye(rank)).max())

    res, _, _ = run_workload(w, 1, on_step=on_step)
    assert_parity(res, "f32", f"geometric {ratio}^-j r{rank} {shapes}")
    # a column of 20000 fp32 roundings: sqrt(m) 2^-24 times a few
    assert max(orth) <= 1e-5
