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


SIDE_BY_SIDE = (1, 2, 3, 5, 8, 16, 40, 128, 256)


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
        for kernels in SIDE_BY_SIDE:
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


# with so many kernels side by side these take the tile of 256 x 160, whose place in LDS is 192 rows long: one column block whole and one ragged,
# two, five; one row block, one and a row, three
@pytest.mark.parametrize("M,N,K", [(256, 160, 264), (257, 304, 520), (700, 312, 264), (500, 808, 520)])
def test_gemm_tile_of_160_columns(M, N, K):
    assert (256, 160) in {C.cephalo_gemm_rows_tile(M, N, K, kernels) for kernels in SIDE_BY_SIDE}
    test_gemm_tiles_give_the_same_bits(M, N, K)


@pytest.mark.parametrize("rows", [1, 7, 64, 65, 200, 4099])
@pytest.mark.parametrize("N", [8, 72, 264, 1032])
@pytest.mark.parametrize("bf16", [False, True])
def test_column_sums_edges(rows, N, bf16):
    """Chunks of 64 rows, 64 vectors of 16 bytes per block; the reduction over 1 to 65 chunks."""
    g = torch.Generator(device="cuda").manual_seed(rows * 31 + N)
    X = torch.randn(rows, N, device="cuda", generator=g)
    X = X.bfloat16() if bf16 else X
    dt = C.BF16 if bf16 else C.F32
    ws = torch.empty(C.cephalo_op_colsum_workspace(rows, N), dtype=torch.uint8, device="cuda").fill_(255)
    out = torch.full((N,), float("nan"), device="cuda")
    C.cephalo_op_colsum(dt, X, rows, N, out, 0.5, 0, ws)
    x = X.double().cpu().numpy()
    bound = (rows + 4) * 2.0 ** -24 * np.abs(x).sum(0)
    assert (np.abs(out.double().cpu().numpy() - 0.5 * x.sum(0)) <= 0.5 * bound).all()
    C.cephalo_op_colsum(dt, X, rows, N, out, 1.0, 1, ws)
    assert (np.abs(out.double().cpu().numpy() - 1.5 * x.sum(0)) <= 1.5 * bound + 2.0 ** -23 * np.abs(x.sum(0))).all()


@pytest.mark.parametrize("rows,N,bf16", [(4096, 32768, True), (4097, 32776, True), (2048, 32768, False), (3001, 32776, False), (40001, 2048, False)])
def test_column_sums_around_the_size_of_the_cache(rows, N, bf16):
    """The blocks' order changes at 256 MB; odd numbers of blocks leave the eight runs of different lengths."""
    g = torch.Generator(device="cuda").manual_seed(rows)
    X = torch.randn(rows, N, device="cuda", generator=g)
    X = X.bfloat16() if bf16 else X
    ws = torch.empty(C.cephalo_op_colsum_workspace(rows, N), dtype=torch.uint8, device="cuda").fill_(255)
    out = torch.full((N,), float("nan"), device="cuda")
    C.cephalo_op_colsum(C.BF16 if bf16 else C.F32, X, rows, N, out, 1.0, 0, ws)
    ref, size = X.sum(0, dtype=torch.float64), X.abs().sum(0, dtype=torch.float64)
    assert ((out.double() - ref).abs() <= (rows + 4) * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("m,S", [(8, 512), (8, 513), (1, 9), (3, 43)])
def test_bias_gradient_of_the_last_projection_is_the_column_sum_of_dy(m, S, bf16):
    """fp32: up to 4096 rows are their own partial sums, more go through the column-sum kernel; bf16: summed in the copy kernel, 32 rows
    per block."""
    H, F = 64, 72
    desc = C.layer_desc(H, 1, F, S, True, C.BF16 if bf16 else C.F32)
    g = torch.Generator(device="cuda").manual_seed(m * S)
    flat = (torch.randn(C.cephalo_layer_param_count(desc), device="cuda", generator=g) * 0.02).to(torch.bfloat16 if bf16 else torch.float32)
    x, dy = torch.randn(m, S, H, device="cuda", generator=g), torch.randn(m, S, H, device="cuda", generator=g)
    y, dx, G = torch.empty_like(x), torch.empty_like(x), torch.full((flat.numel(),), float("nan"), device="cuda")
    sv, sc = C.cephalo_layer_workspace_bytes(desc, m)
    save, scratch = torch.empty(sv, dtype=torch.uint8, device="cuda"), torch.empty(sc, dtype=torch.uint8, device="cuda").fill_(255)
    C.cephalo_layer_fwd(desc, flat, x, y, m, save, scratch)
    C.cephalo_layer_bwd(desc, flat, x, dy, dx, m, save, G, 0.25, 0, scratch)
    off = C.cephalo_layer_param_offsets(desc)[11]
    d = dy.double().cpu().numpy().reshape(-1, H)
    got = G[off:off + H].double().cpu().numpy()
    assert (np.abs(got - 0.25 * d.sum(0)) <= 0.25 * (m * S + 4) * 2.0 ** -24 * np.abs(d).sum(0)).all()
    assert torch.isfinite(G).all() and torch.isfinite(dx).all()


def test_bias_sums_of_two_projections_that_do_not_fit_the_work_area_together():
    """256 wide over 12288 tokens: the weight gradients run one by one in 8 pieces each, and the first bias's pieces leave no room for the
    second's, so they are added before the second GEMM runs."""
    import dataclasses
    from tests import harness as Hn
    from tests.test_wgrad_group import layer_choice
    from workloads import CONFIGS, draw_activations, draw_layer_params
    cfg = dataclasses.replace(CONFIGS["c2"], hidden=256, heads=4, mlp=1024, seq=512, micro_batch=8, n_micro=3)
    tile, pieces = layer_choice(cfg.hidden, cfg.mlp, cfg.batch_share * cfg.seq)
    assert tile == -1 and pieces[1] == 8 and pieces[3] == 8
    tensors = draw_layer_params(cfg, perturbed=True)
    x, dy = draw_activations(cfg)
    Hn.compare_share(cfg, Hn.gpu_share_step(cfg, tensors, x, dy), Hn.oracle_share_step(cfg, tensors, x, dy))


# tokens, out features, in features: every tile of the weight gradient (128 x 128 with four and with two stages, 256 x 128, 256 x 256), ragged
# edges, one slab and less, a token axis in 1, 2, 4 and 8 pieces; the last: on an eighth of the chip and less, 2048 and 136
# of its rows in two launches where no bias gradient comes along, which has the same bits
@pytest.mark.parametrize("T,N,K", [(1, 8, 8), (65, 136, 72), (200, 264, 392), (300, 1544, 1032), (130, 3080, 2056), (4100, 264, 136), (9000, 520, 264), (2100, 1032, 520), (1100, 2184, 1000)])
def test_weight_gradient_tiles(T, N, K):
    print("wgrad tiles", T, N, K, flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + N + K)
    dY, X = torch.randn(T, N, device="cuda", generator=g).bfloat16(), torch.randn(T, K, device="cuda", generator=g).bfloat16()
    a, b = dY.double().cpu().numpy(), X.double().cpu().numpy()
    ref, bound = a.T @ b, _sum_bound(a.T, b, T, 12)
    gref, gbound = a.sum(0), (T + 12) * 2.0 ** -24 * np.abs(a).sum(0)
    ws = torch.empty(C.binding.cephalo_op_linear_wgrad_bias_workspace(C.BF16, T, N, K), dtype=torch.uint8, device="cuda").fill_(255)
    first = None
    before = C.binding.cephalo_gemm_side_by_side(1)
    try:
        for kernels in (1, 2, 3, 5, 8, 16, 256):      # (steers the tile, not the pieces: same bits)
            C.binding.cephalo_gemm_side_by_side(kernels)
            G, gb = torch.full((N, K), float("nan"), device="cuda"), torch.full((N,), float("nan"), device="cuda")
            C.binding.cephalo_op_linear_wgrad_bias(C.BF16, dY, X, T, N, K, G, gb, 1.0, 0, ws)
            assert (np.abs(gb.double().cpu().numpy() - gref) <= gbound).all()
            G2 = torch.full((N, K), float("nan"), device="cuda")
            C.binding.cephalo_op_linear_wgrad(C.BF16, dY, X, T, N, K, G2, 1.0, 0, ws)
            assert torch.equal(G, G2)
            assert first is None or torch.equal(first, G), kernels
            first = G
    finally:
        C.binding.cephalo_gemm_side_by_side(before)
    assert (np.abs(first.double().cpu().numpy() - ref) <= bound).all()


def _attention64(qkv, dO, m, S, A, d, causal, bounds=False):
    """O, (dQ | dK | dV) and lse in 64 bits; bounds: also the rounding error of each that bf16 operands of the second products and bf16 results
    allow, element by element."""
    q, k, v = [t.reshape(m, S, A, d).transpose(1, 2).contiguous().requires_grad_(True) for t in qkv.double().view(m * S, 3, A * d).unbind(1)]
    z = torch.matmul(q, k.transpose(-1, -2).contiguous()) / d ** 0.5
    if causal:
        z = z.masked_fill(torch.ones(S, S, dtype=torch.bool, device=z.device).triu(1), float("-inf"))
    p = torch.softmax(z, -1)
    o = torch.matmul(p, v)
    do = dO.double().view(m, S, A, d).transpose(1, 2).contiguous()
    o.backward(do)
    flat = lambda t: t.transpose(1, 2).reshape(m * S, A * d)
    out = flat(o.detach()), torch.cat([flat(q.grad), flat(k.grad), flat(v.grad)], 1), torch.logsumexp(z, -1).detach()
    if not bounds:
        return out
    # u: rounding to bf16 (8 significant bits).  w: what the fp32 scores, the row sums and the hardware exponential leave in a probability,
    # relative; a score of normal values over d <= 128 terms is off by up to 2^-24 d sum|q||k| / sqrt(d), about 2^-14.
    u, w = 2.0 ** -8, 2.0 ** -13
    with torch.no_grad():
        mm = lambda a, b: torch.matmul(a, b.contiguous())
        q, k, v, o, t = q.detach(), k.detach(), v.detach(), o.detach(), p.transpose(-1, -2)
        e_o = u * o.abs() + (u + w) * mm(p, v.abs())
        dp = mm(do, v.transpose(-1, -2)) - (do * o).sum(-1, keepdim=True)
        e_s = (u + w) * p * dp.abs() + p * ((do.abs() * e_o).sum(-1, keepdim=True) + w * mm(do.abs(), v.abs().transpose(-1, -2)))
        e_q = mm(e_s, k.abs()) / d ** 0.5
        e_k = mm(e_s.transpose(-1, -2).contiguous(), q.abs()) / d ** 0.5
        e_v = (u + w) * mm(t.contiguous(), do.abs())
    return out + (flat(e_o), torch.cat([flat(e_q), flat(e_k), flat(e_v)], 1) + u * out[1].abs())


# head widths: the 32-, 64- and 128-wide tiles, full and narrower; tokens around the 32-, 64- and 128-token pieces; the last column: few tiles
# (one per block) or more than 256 of them (a tile and its mirror image per block under the causal mask, with an odd and an even count)
@pytest.mark.parametrize("d", [8, 32, 40, 64, 72, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("m,S,A", [(1, 1, 1), (3, 31, 2), (1, 65, 3), (2, 129, 2), (1, 300, 90), (2, 450, 34)])
def test_attention_tiles(m, S, A, d, causal):
    print("attention tiles", m, S, A, d, causal, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m * S + d)
    H = A * d
    qkv, dO = torch.randn(m * S, 3 * H, device="cuda", generator=g).bfloat16(), torch.randn(m * S, H, device="cuda", generator=g).bfloat16()
    ro, rg, rl, bo, bg = _attention64(qkv, dO, m, S, A, d, causal, bounds=True)
    desc = C.layer_desc(H, A, 4 * H, S, causal, C.BF16)
    O = torch.full((m * S, H), float("nan"), device="cuda", dtype=torch.bfloat16)
    lse, dvec = torch.full((m, A, S), float("nan"), device="cuda"), torch.full((m, A, S), float("nan"), device="cuda")
    dqkv = torch.full((m * S, 3 * H), float("nan"), device="cuda", dtype=torch.bfloat16)
    C.cephalo_op_attention_fwd(desc, qkv, O, lse, m)
    C.cephalo_op_attention_bwd(desc, qkv, O, dO, lse, dvec, dqkv, m)

    for what, got, ref, bound in [("O", O, ro, bo)] + [(n, dqkv[:, i * H:(i + 1) * H], rg[:, i * H:(i + 1) * H], bg[:, i * H:(i + 1) * H]) for i, n in enumerate(("dQ", "dK", "dV"))]:
        e = (got.double() - ref).abs()
        print("  %s: %.2f of the bound, %.1e of the largest element" % (what, (e / (bound + 1e-12)).max(), e.max() / (ref.abs().max() + 1e-12)), flush=True)
        assert (e <= bound + 1e-12).all(), what
    assert (lse.double() - rl).abs().max() < 2e-3
    dv = (dO.double() * O.double()).view(m, S, A, d).sum(-1).transpose(1, 2)
    assert (dvec.double() - dv).abs().max() <= (d + 4) * 2.0 ** -24 * (dO.double() * O.double()).abs().view(m, S, A, d).sum(-1).max()


@pytest.mark.parametrize("H,heads,S,b", [(320, 5, 150, 4), (64, 1, 1, 1), (256, 4, 33, 1), (264, 3, 700, 4), (8, 1, 33, 1000)])
@pytest.mark.parametrize("spread", ["few", "many", "one"])
def test_token_embedding_gradient(H, heads, S, b, spread):
    """Rows of 1 to 2 wavefronts; runs of equal ids inside a segment of 32, across several, and of all tokens; 1 to 2800 tokens ranked by
    counting, 33000 sorted by the network."""
    V = {"few": 13, "many": 4096, "one": 5}[spread]
    desc = C.layer_desc(H, heads, 72, S, True, C.BF16, kind=C.LAYER_LLAMA)
    sd = C.StackDesc(desc, 1, V, 0, 0, 0)
    g = torch.Generator(device="cuda").manual_seed(H + S)
    P = C.cephalo_stack_param_count(sd)
    flat = (torch.randn(P, device="cuda", generator=g) * 0.02).bfloat16()
    ids = torch.randint(0, V, (b, S), device="cuda", generator=g, dtype=torch.int32)
    if spread == "one":
        ids.fill_(3)
    targets = torch.randint(0, V, (b, S), device="cuda", generator=g, dtype=torch.int32)
    G, loss = torch.full((P,), float("nan"), device="cuda"), torch.empty(1, device="cuda")
    m = 500 if b == 1000 else 1
    ws = torch.empty(C.cephalo_stack_workspace_bytes(sd, b, m), dtype=torch.uint8, device="cuda")
    C.cephalo_stack_step(sd, flat, ids, targets, b, m, G, 64.0, loss, ws)
    at = C.binding.cephalo_stack_workspace_regions(sd, b, m)[1]
    n = b * S
    dx0 = ws[at:at + 4 * n * H].view(torch.float32).view(n, H).double()
    rows = ids.view(-1).long()
    ref = torch.zeros(V, H, dtype=torch.float64, device="cuda").index_add_(0, rows, dx0)
    size = torch.zeros(V, H, dtype=torch.float64, device="cuda").index_add_(0, rows, dx0.abs())
    got = G[:V * H].view(V, H).double()
    assert torch.isfinite(G).all() and dx0.abs().max() > 0
    assert ((got - ref).abs() <= n * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("d", [4, 20, 30, 32, 64, 100, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("m,S,A", [(1, 1, 2), (2, 15, 4), (1, 17, 2), (2, 64, 2), (1, 150, 4)])
def test_fp32_attention_edges(m, S, A, d, causal):
    """Blocks of 16 queries and keys over four wavefronts, head widths between the 32-, 64- and 128-wide forms, a width that takes scalar loads."""
    print("attention f32", m, S, A, d, causal, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m * S + d)
    H = A * d
    qkv, dO = torch.randn(m * S, 3 * H, device="cuda", generator=g), torch.randn(m * S, H, device="cuda", generator=g)
    ro, rg, rl = _attention64(qkv, dO, m, S, A, d, causal)
    desc = C.layer_desc(H, A, 4 * H, S, causal, C.F32)
    O, lse, dvec = torch.full((m * S, H), float("nan"), device="cuda"), torch.full((m, A, S), float("nan"), device="cuda"), torch.full((m, A, S), float("nan"), device="cuda")
    dqkv = torch.full((m * S, 3 * H), float("nan"), device="cuda")
    C.cephalo_op_attention_fwd(desc, qkv, O, lse, m)
    C.cephalo_op_attention_bwd(desc, qkv, O, dO, lse, dvec, dqkv, m)
    # fp32 sums over up to S + d terms of size about 1, scores of size sqrt(d): 2^-24 (S + d) sqrt(d) with a margin of 4
    tol = 4 * 2.0 ** -24 * (S + d) * d ** 0.5
    for got, ref in ((O, ro), (lse, rl), (dqkv, rg)):
        assert (got.double() - ref).abs().max() <= tol * max(1.0, ref.abs().max().item())


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_fp32_attention_masked_tokens_stay_out(bad):
    """Under the causal mask a token's values reach no earlier token's output, whatever they are."""
    m, S, A, d = 1, 37, 2, 64
    H = A * d
    g = torch.Generator(device="cuda").manual_seed(5)
    qkv = torch.randn(m * S, 3 * H, device="cuda", generator=g)
    desc = C.layer_desc(H, A, 4 * H, S, True, C.F32)
    clean, lse = torch.empty(m * S, H, device="cuda"), torch.empty(m, A, S, device="cuda")
    C.cephalo_op_attention_fwd(desc, qkv, clean, lse, m)
    for at in (36, 20, 16):
        dirty = qkv.clone()
        dirty[at, 2 * H + 3] = bad
        out = torch.empty_like(clean)
        C.cephalo_op_attention_fwd(desc, dirty, out, lse, m)
        assert torch.isfinite(out[:at]).all() and (out[:at] - clean[:at]).abs().max() < 1e-5
        assert not torch.isfinite(out[at:, 3]).any()


@pytest.mark.parametrize("H", [8, 256, 512, 520, 1024, 1032, 2048, 2056, 4096])
@pytest.mark.parametrize("rows", [1, 8, 13, 100])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("rms", [False, True])
def test_norm_backward_teams(rows, H, bf16, rms):
    """Teams of 64, 128 and 256 threads per row with 1, 2 and 4 vectors each, around the widths where they change; blocks of 8 rows, partly filled."""
    g = torch.Generator(device="cuda").manual_seed(rows + H)
    du, x, res = (torch.randn(rows, H, device="cuda", generator=g) for _ in range(3))
    dt = torch.bfloat16 if bf16 else torch.float32
    gam = (1 + 0.1 * torch.randn(H, device="cuda", generator=g)).to(dt)
    x64, d64, g64 = x.double(), du.double(), gam.double()
    mean = torch.zeros(rows, device="cuda", dtype=torch.float64) if rms else x64.mean(1)
    rstd = 1 / torch.sqrt(((x64 - mean[:, None]) ** 2).mean(1) + 1e-5)
    mean, rstd = mean.float(), rstd.float()
    xh = (x64 - mean.double()[:, None]) * rstd.double()[:, None]
    gg = d64 * g64
    ref = res.double() + rstd.double()[:, None] * (gg - (0 if rms else gg.mean(1, keepdim=True)) - xh * (gg * xh).mean(1, keepdim=True))
    dx, dg, db = torch.full_like(x, float("nan")), torch.full((H,), float("nan"), device="cuda"), torch.full((H,), float("nan"), device="cuda")
    low = torch.full((rows, H), float("nan"), device="cuda", dtype=dt) if bf16 else None
    ws = torch.empty(max(C.cephalo_op_norm_bwd_workspace(rows, H), C.binding.cephalo_op_norm_bwd_sums_workspace(rows, H)), dtype=torch.uint8, device="cuda").fill_(255)
    C.cephalo_op_norm_bwd(C.BF16 if bf16 else C.F32, rms, du, x, mean, rstd, gam, res, dx, low, dg, None if rms else db, rows, H, ws)
    eps = 2.0 ** -24
    # sums over H terms of size |g| and |g xhat|, then a handful of roundings of values up to the largest of the row
    size = res.abs().double() + rstd.double()[:, None] * (gg.abs() + gg.abs().mean(1, keepdim=True) + xh.abs() * (gg * xh).abs().mean(1, keepdim=True))
    assert ((dx.double() - ref).abs() <= (H + 16) * eps * size).all()
    if bf16:
        assert torch.equal(low, dx.bfloat16())
    assert ((dg.double() - (d64 * xh).sum(0)).abs() <= (rows + 8) * eps * (d64 * xh).abs().sum(0) + 1e-30).all()
    if not rms:
        assert ((db.double() - d64.sum(0)).abs() <= (rows + 8) * eps * d64.abs().sum(0)).all()
        ds, dx2, dg2, db2 = torch.full((H,), float("nan"), device="cuda"), torch.empty_like(dx), torch.empty_like(dg), torch.empty_like(db)
        C.binding.cephalo_op_norm_bwd_sums(C.BF16 if bf16 else C.F32, du, x, mean, rstd, gam, res, dx2, low, dg2, db2, ds, rows, H, ws)
        assert torch.equal(dx, dx2) and torch.equal(dg, dg2) and torch.equal(db, db2)
        assert ((ds.double() - dx.double().sum(0)).abs() <= (rows + 8) * eps * dx.double().abs().sum(0)).all()
