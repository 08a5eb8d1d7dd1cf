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


# rows, columns, contraction: every tile of the k-contiguous products (64 x 64 up to 256 x 256) with ragged edges; a contraction shorter
# than a slab of 64, of one slab, of an odd number of slabs, and one with a remainder
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (65, 72, 64), (130, 200, 72), (257, 264, 320), (300, 1032, 456), (1000, 1544, 192), (2050, 2056, 136), (1550, 400, 136),
                                   (450, 1624, 264), (550, 2576, 520)])
def test_gemm_tiles_give_the_same_bits(M, N, K):
    """The number of kernels side by side steers the tile choice; each tile adds the products of an output in the same order."""
    print("gemm tiles", M, N, K, flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    X = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    W = (torch.randn(N, K, device="cuda", generator=g) * 0.05).bfloat16()
    b = torch.randn(N, device="cuda", generator=g).bfloat16()
    R = torch.randn(M, N, device="cuda", generator=g)
    acc = X.double().cpu().numpy() @ W.double().cpu().numpy().T
    bound = _sum_bound(X.double().cpu().numpy(), W.double().cpu().numpy().T, K)
    first = {}
    before = C.binding.cephalo_gemm_side_by_side(1)
    try:
        for kernels in (1, 2, 3, 5, 8, 16, 40, 128, 256):
            C.binding.cephalo_gemm_side_by_side(kernels)
            out = torch.full((M, N), float("nan"), device="cuda")
            C.cephalo_op_gemm(C.BF16, X, K, 1, W, K, 1, M, N, K, C.EPI_NONE_F32, C=out)
            res = torch.full((M, N), float("nan"), device="cuda")
            C.cephalo_op_gemm(C.BF16, X, K, 1, W, K, 1, M, N, K, C.EPI_BIAS_RESID_F32, C=res, bias=b, R=R)
            h = torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
            d = torch.full((M, N), float("nan"), device="cuda", dtype=torch.float16)
            C.cephalo_op_gemm(C.BF16, X, K, 1, W, K, 1, M, N, K, C.EPI_BIAS_GELU_DERIV, C=h, bias=b, Z=d)
            mul = torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
            C.cephalo_op_gemm(C.BF16, X, K, 1, W, K, 1, M, N, K, C.EPI_MUL, C=mul, Z=d)
            for name, t in (("plain", out), ("resid", res), ("gelu", h), ("deriv", d), ("mul", mul)):
                if name in first:
                    assert torch.equal(first[name], t), (name, kernels)
                else:
                    first[name] = t
    finally:
        C.binding.cephalo_gemm_side_by_side(before)
    assert (np.abs(first["plain"].double().cpu().numpy() - acc) <= bound).all()
    ref = acc + b.double().cpu().numpy() + R.double().cpu().numpy()
    assert (np.abs(first["resid"].double().cpu().numpy() - ref) <= bound + 3 * 2.0 ** -24 * (np.abs(acc) + np.abs(ref) + 4)).all()
