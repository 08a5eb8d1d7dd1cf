"""GPU parity of attention forward/backward (plain fp32 kernel and matrix-core bf16 kernel)
against the oracle's definition, on the packed [tokens, 3H] projection layout."""
import numpy as np
import pytest
import torch

import paper_2411_01075_amd as C
from oracle import layer as olayer
from oracle.precision import round_to_bf16
from tests.harness import rel_errors

pytestmark = pytest.mark.gpu

CASES = [  # bf16?, m, S, heads, head dim, causal
    (True, 2, 256, 2, 64, True),
    (True, 1, 200, 3, 64, False),      # ragged: S not a multiple of the 64/128 tiles
    (True, 2, 333, 2, 128, True),
    (True, 1, 128, 1, 128, False),
    (True, 1, 40, 2, 64, True),        # shorter than one tile
    (True, 1, 1024, 2, 64, True),
    # head widths between the 64- and 128-wide tiles (the paper's model table has 32, 104 and 112 among others)
    (True, 2, 200, 3, 32, True),
    (True, 1, 333, 2, 104, True),
    (True, 2, 197, 2, 112, False),
    (True, 1, 150, 5, 8, True),
    (True, 1, 260, 2, 96, False),
    (True, 1, 130, 3, 40, False),
    # the 128-wide causal forward (two wavefront groups in turns): a single tile, an even tile count, a narrow head on the wide tile
    (True, 1, 100, 2, 128, True),
    (True, 2, 256, 2, 128, True),
    (True, 1, 300, 2, 72, True),
    (True, 1, 640, 1, 128, True),
    (False, 2, 70, 3, 24, True),
    (False, 1, 128, 2, 64, False),
]


def oracle_attention(qkv, dO, m, S, A, d, causal):
    H = A * d
    t = qkv.reshape(m, S, 3 * H)
    q, k, v = (olayer.split_heads(t[..., i * H:(i + 1) * H], A) for i in range(3))
    Oh, P = olayer.attention_fwd(q, k, v, causal)
    # log-sum-exp of the scaled, masked scores
    Z = (q @ k.transpose(0, 1, 3, 2)) / np.sqrt(d)
    if causal:
        Z = np.where(np.triu(np.ones((S, S), dtype=bool), 1), -np.inf, Z)
    zmax = Z.max(-1, keepdims=True)
    lse = (zmax + np.log(np.exp(Z - zmax).sum(-1, keepdims=True)))[..., 0]
    dQ, dK, dV = olayer.attention_bwd(olayer.split_heads(dO.reshape(m, S, H), A), q, k, v, P)
    dqkv = np.concatenate([olayer.merge_heads(g) for g in (dQ, dK, dV)], axis=-1).reshape(m * S, 3 * H)
    return olayer.merge_heads(Oh).reshape(m * S, H), lse, dqkv


@pytest.mark.parametrize("bf16,m,S,A,d,causal", CASES)
def test_attention_fwd_bwd(bf16, m, S, A, d, causal):
    print("attention", bf16, m, S, A, d, causal, flush=True)
    H = A * d
    rng = np.random.default_rng(S + d)
    qkv = rng.standard_normal((m * S, 3 * H)).astype(np.float32)
    dO = rng.standard_normal((m * S, H)).astype(np.float32)
    rnd = round_to_bf16 if bf16 else (lambda a: a.astype(np.float64))
    O_ref, lse_ref, dqkv_ref = oracle_attention(rnd(qkv), rnd(dO), m, S, A, d, causal)
    dt = torch.bfloat16 if bf16 else torch.float32
    desc = C.layer_desc(H, A, 4 * H, S, causal, C.BF16 if bf16 else C.F32)
    dqkv_in = torch.from_numpy(qkv).cuda().to(dt)
    ddO = torch.from_numpy(dO).cuda().to(dt)
    O = torch.full((m * S, H), float("nan"), dtype=dt, device="cuda")
    lse = torch.full((m, A, S), float("nan"), dtype=torch.float32, device="cuda")
    C.cephalo_op_attention_fwd(desc, dqkv_in, O, lse, m)
    torch.cuda.synchronize()
    tol_max, tol_mean = (2e-2, 5e-3) if bf16 else (1e-4, 1e-4)
    e = rel_errors(O.double().cpu().numpy(), O_ref)
    print("O", e, flush=True)
    assert e[0] < tol_max and e[1] < tol_mean
    assert np.max(np.abs(lse.double().cpu().numpy() - lse_ref)) < (2e-3 if bf16 else 1e-4)
    dvec = torch.empty((m, A, S), dtype=torch.float32, device="cuda")
    dqkv = torch.full((m * S, 3 * H), float("nan"), dtype=dt, device="cuda")
    C.cephalo_op_attention_bwd(desc, dqkv_in, O, ddO, lse, dvec, dqkv, m)
    torch.cuda.synchronize()
    got = dqkv.double().cpu().numpy()
    for name, sl in (("dQ", slice(0, H)), ("dK", slice(H, 2 * H)), ("dV", slice(2 * H, 3 * H))):
        e = rel_errors(got[:, sl], dqkv_ref[:, sl])
        print(name, e, flush=True)
        assert e[0] < tol_max and e[1] < tol_mean, name


def _two_halves(q, k, v):
    """The causal forward of one sample [heads, S, d] in 64 bits but for the probabilities: rounded to bf16 relative to the running maximum of their half
    of the keys (tiles of 64, even or odd), which is raised where some row of a block of 32 queries would see an exponent above 8."""
    A, S, d = q.shape
    z2 = torch.full((A, S, S), float("-inf"), device=q.device, dtype=torch.float64)
    seen = torch.ones(S, S, dtype=torch.bool, device=q.device).tril()
    z2[:, seen] = (torch.matmul(q.double(), k.double().transpose(1, 2).contiguous()) * (d ** -0.5 * 1.4426950408889634))[:, seen]
    out = torch.empty(A, S, d, device=q.device, dtype=torch.float64)
    for q0 in range(0, S, 32):
        rows, halves = slice(q0, min(S, q0 + 32)), []
        for parity in (0, 1):
            m, l = (torch.full((A, rows.stop - q0, 1), x, device=q.device, dtype=torch.float64) for x in (float("-inf"), 0.0))
            o = torch.zeros(A, rows.stop - q0, d, device=q.device, dtype=torch.float64)
            for t0 in range(64 * parity, rows.stop, 128):
                z = z2[:, rows, t0:t0 + 64]
                mx = z.max(-1, keepdim=True).values
                raised = torch.maximum(m, mx)
                up = (mx > m + 8).flatten(1).any(1)[:, None, None]
                new = torch.where(up, raised, m)
                alpha = torch.where(torch.isinf(new), torch.ones_like(new), torch.exp2(m - new))
                l, o, m = l * alpha, o * alpha, new
                p = torch.exp2(z - torch.where(torch.isinf(m), torch.zeros_like(m), m))
                l, o = l + p.sum(-1, keepdim=True), o + torch.matmul(p.to(torch.bfloat16).double(), v[:, t0:t0 + 64].double().contiguous())
            halves.append((m, l, o))
        top = torch.maximum(halves[0][0], halves[1][0])
        w = [torch.where(torch.isinf(m), torch.zeros_like(m), torch.exp2(m - top)) for m, _, _ in halves]
        out[:, rows] = (halves[0][2] * w[0] + halves[1][2] * w[1]) / (halves[0][1] * w[0] + halves[1][1] * w[1])
    return out


@pytest.mark.parametrize("S,A,d,spread", [(1100, 9, 64, 1.0), (1100, 9, 64, 5.0), (700, 12, 32, 2.25), (1000, 10, 48, 2.25)])      # (spread: standard deviation of the scores)
def test_probabilities_are_rounded_relative_to_the_maximum_of_their_half(S, A, d, spread):
    print("attention halves", S, A, d, spread, flush=True)
    H = A * d
    g = torch.Generator(device="cuda").manual_seed(S)
    qkv = torch.randn(S, 3 * H, device="cuda", generator=g)
    qkv[:, :2 * H] *= spread ** 0.5
    qkv = qkv.to(torch.bfloat16)
    O, lse = torch.full((S, H), float("nan"), dtype=torch.bfloat16, device="cuda"), torch.empty(1, A, S, device="cuda")
    C.cephalo_op_attention_fwd(C.layer_desc(H, A, 4 * H, S, True, C.BF16), qkv, O, lse, 1)
    q, k, v = (qkv[:, i * H:(i + 1) * H].reshape(S, A, d).transpose(0, 1).contiguous() for i in range(3))
    want = _two_halves(q, k, v).transpose(0, 1).reshape(S, H).to(torch.bfloat16).double()
    e = float((O.double() - want).norm() / want.norm())
    print("difference %.2e" % e, flush=True)
    # Results that fall near the middle between two bf16 values are rounded apart by fp32's errors (2^-8 of a value, of one in a few hundred), and so are probabilities.
    # Relative to one maximum of all keys the probabilities' rounding errors are others: 1.5e-3 and more.
    assert e <= 4e-4


@pytest.mark.parametrize("m,S,A,d", [
    (20, 300, 5, 64),       # 100 heads, 300 tiles: forward with four wavefronts, by head, some XCDs with one head more; backward in one launch by head
    (8, 520, 13, 32),       # 520 tiles, 13 heads an XCD: two launches by head
    (6, 700, 15, 64),       # 540 tiles, 90 heads: two launches by head, some XCDs with one head more
    (4, 1100, 9, 64),       # 324 tiles of long samples: forward with eight wavefronts, in pairs, an odd number of tiles
    (9, 2100, 3, 64),       # 459 tiles: backward in one launch in pairs, the statistics in two windows
    (1, 2100, 3, 32),       # 51 tiles: single ones, in two windows
    (4, 4200, 5, 32),       # 660 tiles of 20 heads
    (3, 4200, 3, 64),       # 297 tiles of 9 heads: no by head
    (5, 700, 9, 128),       # pairs, heads of 128
    (64, 64, 8, 64),        # one tile a head
])
def test_causal_samples_do_not_depend_on_the_launch(m, S, A, d):
    """The order of the tiles follows from the launch's size; a sample's results are the same bits as by itself."""
    print("attention order", m, S, A, d, flush=True)
    H = A * d
    g = torch.Generator(device="cuda").manual_seed(S)
    qkv = torch.randn(m * S, 3 * H, device="cuda", generator=g).to(torch.bfloat16)
    dO = torch.randn(m * S, H, device="cuda", generator=g).to(torch.bfloat16)
    desc = C.layer_desc(H, A, 4 * H, S, True, C.BF16)

    def run(qkv, dO, m):
        O, dqkv = torch.full_like(dO, float("nan")), torch.full_like(qkv, float("nan"))
        lse, dvec = (torch.full((m, A, S), float("nan"), device="cuda") for _ in range(2))
        C.cephalo_op_attention_fwd(desc, qkv, O, lse, m)
        C.cephalo_op_attention_bwd(desc, qkv, O, dO, lse, dvec, dqkv, m)
        return O, lse, dqkv

    O, lse, dqkv = run(qkv, dO, m)
    assert not any(torch.isnan(t).any() for t in (O, lse, dqkv))
    for n in range(m):
        rows = slice(n * S, (n + 1) * S)
        o1, l1, g1 = run(qkv[rows].contiguous(), dO[rows].contiguous(), 1)
        assert torch.equal(o1, O[rows]) and torch.equal(l1[0], lse[n]) and torch.equal(g1, dqkv[rows]), n


@pytest.mark.parametrize("S,A,d,causal", [
    (40, 8, 64, True),          # under one tile
    (64, 6, 32, False),
    (197, 12, 64, False),
    (333, 10, 64, True),
    (640, 5, 24, True),
    (640, 5, 64, False),
    (2048, 2, 64, False),       # the longest sample whose statistics the one launch holds at once
    (2048, 1, 32, True),
    (2049, 2, 64, False),       # one row beyond it
    (4160, 1, 64, True),        # three windows of statistics
])
def test_backward_in_one_launch_or_two(S, A, d, causal):
    """Up to 512 tiles, or 384 of more than four a head without a mask, the backward of narrow heads is one launch; a sample's results are the same bits on both sides."""
    print("attention backward launches", S, A, d, causal, flush=True)
    H, limit, each = A * d, 512 if causal or S <= 512 else 384, A * ((S + 127) // 128)
    below = max(1, limit // each)                                        # samples of the last launch in one, the first in two
    m = below + 1
    g = torch.Generator(device="cuda").manual_seed(S + d)
    qkv = torch.randn(m * S, 3 * H, device="cuda", generator=g).to(torch.bfloat16)
    dO = torch.randn(m * S, H, device="cuda", generator=g).to(torch.bfloat16)
    desc = C.layer_desc(H, A, 4 * H, S, causal, C.BF16)
    O, lse = torch.empty_like(dO), torch.empty(m, A, S, device="cuda")
    C.cephalo_op_attention_fwd(desc, qkv, O, lse, m)

    def backward(n):
        dqkv, dvec = torch.full((n * S, 3 * H), float("nan"), dtype=torch.bfloat16, device="cuda"), torch.empty(n, A, S, device="cuda")
        C.cephalo_op_attention_bwd(desc, qkv[:n * S], O[:n * S], dO[:n * S], lse[:n], dvec, dqkv, n)
        return dqkv

    many, most, one = backward(m), backward(below), backward(1)
    assert not torch.isnan(many).any()
    assert torch.equal(most, many[:below * S]) and torch.equal(one, many[:S])


@pytest.mark.parametrize("S,A,d,causal", [(1, 4, 64, True), (37, 3, 24, True), (130, 4, 64, False), (200, 2, 30, True), (260, 2, 128, True), (100, 3, 100, False)])
def test_fp32_backward_in_one_launch_or_two(S, A, d, causal):
    """Up to 512 blocks (256 for heads wider than 64) the fp32 backward is one launch; a sample's results are the same bits on both sides."""
    print("fp32 attention backward launches", S, A, d, causal, flush=True)
    H, limit, each = A * d, 512 if d <= 64 else 256, 2 * A * ((S + 15) // 16)
    below = limit // each
    m = below + 1
    g = torch.Generator(device="cuda").manual_seed(S + d)
    qkv, dO = torch.randn(m * S, 3 * H, device="cuda", generator=g), torch.randn(m * S, H, device="cuda", generator=g)
    desc = C.layer_desc(H, A, 4 * H, S, causal, C.F32)
    O, lse = torch.empty_like(dO), torch.empty(m, A, S, device="cuda")
    C.cephalo_op_attention_fwd(desc, qkv, O, lse, m)

    def backward(n):
        dqkv, dvec = torch.full((n * S, 3 * H), float("nan"), device="cuda"), torch.full((n, A, S), float("nan"), device="cuda")
        C.cephalo_op_attention_bwd(desc, qkv[:n * S], O[:n * S], dO[:n * S], lse[:n], dvec, dqkv, n)
        return dqkv, dvec

    many, most, one = backward(m), backward(below), backward(1)
    assert not any(torch.isnan(t).any() for t in many)
    for t, (rows, n) in ((most, (below * S, below)), (one, (S, 1))):
        assert torch.equal(t[0], many[0][:rows]) and torch.equal(t[1], many[1][:n])
