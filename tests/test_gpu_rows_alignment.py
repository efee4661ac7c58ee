"""Row-sparse step on rows at any alignment and of any width: P_hat, Q, err and
M_hat are bitwise those of occ_step on the gathered rows (the same tiling, the
same products in the same order), whether the list ends in the matrix's last
row or not.  The unlisted rows of M, err and M_hat and everything between the
rows hold NaN: a value read from there and not dropped shows in every output,
and a write there shows in the buffers.
"""

import pytest

from gpu_util import torch_mod

pytestmark = pytest.mark.gpu


def _placed(x, offset, ld):
    """x (m x n) at element `offset` of a NaN-filled buffer, pitch ld: (view, buffer)."""
    torch = torch_mod()
    m, n = x.shape
    buf = torch.full((offset + m * ld + 64,), float("nan"), dtype=x.dtype, device="cuda")
    view = buf.as_strided((m, n), (ld, 1), offset)
    view.copy_(x)
    return view, buf


def _untouched(view, buf, rows):
    """Everything of `buf` but the given rows of `view` is NaN."""
    torch = torch_mod()
    keep = torch.ones_like(buf, dtype=torch.bool)
    keep.as_strided(view.shape, view.stride(), view.storage_offset())[rows] = False
    return bool(buf[keep].isnan().all())


# widths with whole 32-column steps and 8-column chunks and without; 160 rows:
# one large-rank row tile and a piece of the next
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [3, 16, 17, 48, 128])
@pytest.mark.parametrize("cols", [31, 97, 128, 257, 395, 1000])
def test_rows_equal_step_on_gathered_rows(cols, rank, dtype):
    from paper_2301_09830_amd import optcc
    torch = torch_mod()
    if rank > cols:
        pytest.skip("rank exceeds the matrix")
    vocab, listed = 500, 160
    g = torch.Generator(device="cuda")
    g.manual_seed(cols * 131 + rank)
    order = torch.randperm(vocab - 1, generator=g, device="cuda")
    Q0 = torch.randn((cols, rank), generator=g, device="cuda")
    M = torch.randn((vocab, cols), generator=g, device="cuda")
    M = M.bfloat16() if dtype == "bf16" else M
    err = 0.1 * torch.randn((vocab, cols), generator=g, device="cuda")
    for last in (False, True):
        at = order[:listed].clone()
        if last:
            at[0] = vocab - 1
        at = torch.sort(at)[0]
        off_list = torch.ones(vocab, dtype=torch.bool, device="cuda")
        off_list[at] = False
        Md, ed, Qd = M[at].contiguous(), err[at].contiguous(), Q0.clone()
        Pd, Hd = optcc.occ_step(Md, ed, Qd, rank, 2)
        for off, ld in ((0, (cols + 31) // 32 * 32), (1, cols + 3), (3, cols)):
            Mv, _ = _placed(M, off, ld)
            ev, ebuf = _placed(err, off, ld)
            hv, hbuf = _placed(torch.zeros_like(err), off, ld)
            for v in (Mv, ev, hv):
                v[off_list] = float("nan")
            Qv = Q0.clone()
            Pv, _ = optcc.occ_step_rows(Mv, ev, Qv, at.int(), rank, 2, M_hat=hv)
            torch.cuda.synchronize()
            where = f"cols {cols} r{rank} {dtype} last {last} offset {off} ld {ld}"
            assert torch.equal(Pv, Pd) and torch.equal(Qv, Qd), where
            assert torch.equal(ev[at], ed) and torch.equal(hv[at], Hd), where
            assert _untouched(ev, ebuf, at) and _untouched(hv, hbuf, at), where
