"""Kernels and dispatch branches at the sizes where they can go wrong: tile edges, remainders, unaligned pitches, the smallest and
largest of a range.  References in float64 on the host."""
import numpy as np
import pytest
import torch

import paper_2411_01075_amd as C

pytestmark = pytest.mark.gpu


def _sum_bound(a, b, terms, extra=4):
    """Bound of the rounding error of a fp32 dot product of `terms` terms in any order: (terms + extra) 2^-24 sum |a||b|."""
    return (terms + extra) * 2.0 ** -24 * (np.abs(a) @ np.abs(b))


# (M, N, K, pitch beyond the extent): tiles of 32 x 32, slabs of 128 in pieces of 32; a pitch that is not a multiple of four takes
# the scalar loads
@pytest.mark.parametrize("M,N,K,pad", [(1, 1, 1, 0), (32, 32, 128, 0), (33, 31, 129, 0), (64, 36, 132, 0), (5, 100, 260, 0), (40, 48, 64, 3), (96, 32, 516, 4)])
@pytest.mark.parametrize("layout", ["kk", "kr", "rr", "rk"])
def test_fp32_gemm_edges(M, N, K, pad, layout):
    print("gemm_f32", M, N, K, pad, layout, flush=True)
    rng = np.random.default_rng(M + 3 * N + 7 * K + pad)
    A, B = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)

    def operand(x, kfast):
        y = np.ascontiguousarray(x if kfast else x.T)
        buf = np.full((y.shape[0], y.shape[1] + pad), np.nan, dtype=np.float32)      # what lies in the pitch is never used
        buf[:, :y.shape[1]] = y
        t = torch.from_numpy(buf).cuda()
        return t, (buf.shape[1], 1) if kfast else (1, buf.shape[1])
    ta, (ars, acs) = operand(A, layout[0] == "k")
    tb, (brs, bcs) = operand(B, layout[1] == "k")
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    bound = _sum_bound(A.astype(np.float64), B.astype(np.float64).T, K)
    out = torch.full((M, N), float("nan"), device="cuda")
    C.cephalo_op_gemm(C.F32, ta, ars, acs, tb, brs, bcs, M, N, K, C.EPI_NONE, C=out)
    assert (np.abs(out.double().cpu().numpy() - ref) <= bound).all()
    C.cephalo_op_gemm(C.F32, ta, ars, acs, tb, brs, bcs, M, N, K, C.EPI_GRAD, G=out, scale=1.0, accumulate=1)
    assert (np.abs(out.double().cpu().numpy() - 2 * ref) <= 3 * bound + 2.0 ** -23 * np.abs(ref)).all()
