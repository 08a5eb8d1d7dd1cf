"""Several micro-batches per launch: the share and stack calls give the results of single micro-batches bit for bit, however many
of them a launch takes and whichever stream it runs on."""
import pytest
import torch

import paper_2411_01075_amd as C

pytestmark = pytest.mark.gpu


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device="cuda").fill_(255)      # (work areas start as NaNs)


def _flat(n, dtype):
    g = torch.Generator(device="cuda").manual_seed(5)
    return (torch.randn(n, device="cuda", generator=g) * 0.05).to(torch.float32 if dtype == C.F32 else torch.bfloat16)


def _share(desc, b, m, side=False):
    g = torch.Generator(device="cuda").manual_seed(7)
    x, dy = (torch.randn(b, desc.seq, desc.hidden, device="cuda", generator=g) for _ in range(2))
    flat = _flat(C.cephalo_layer_param_count(desc), desc.dtype)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    G = torch.full((flat.numel(),), float("nan"), device="cuda")
    save, scratch = (_bytes(n) for n in C.cephalo_share_workspace_bytes(desc, b, m))
    if side:
        C.cephalo_share_layer_step_interleaved(desc, flat, x, y, dy, dx, b, m, save, G, 0.5, scratch, torch.cuda.Stream())
    else:
        C.cephalo_share_layer_step(desc, flat, x, y, dy, dx, b, m, save, G, 0.5, scratch)
    torch.cuda.synchronize()
    return flat, x, dy, y, dx, G


@pytest.mark.parametrize("kind,dtype", [("gpt", "bf16"), ("llama", "bf16"), ("gpt", "f32"), ("llama", "f32")])
@pytest.mark.parametrize("S,m,l", [(37, 1, 3), (197, 1, 5), (64, 3, 2), (9, 5, 9)])      # (micro-batches that are no multiple of a norm block's 8 rows)
def test_share_is_its_micro_batches_bit_for_bit(kind, dtype, S, m, l):
    print(kind, dtype, S, m, l, flush=True)
    desc = C.layer_desc(128, 4, 344, S, True, C.F32 if dtype == "f32" else C.BF16, 1e-5, C.LAYER_LLAMA if kind == "llama" else C.LAYER_GPT)
    flat, x, dy, y, dx, G = _share(desc, m * l, m)
    assert not torch.isnan(G).any()
    Gm = torch.full_like(G, float("nan"))
    save, scratch = (_bytes(n) for n in C.cephalo_layer_workspace_bytes(desc, m))
    for j in range(l):
        sl = slice(j * m, (j + 1) * m)
        yj, dxj = torch.empty_like(x[sl]), torch.empty_like(x[sl])
        C.cephalo_layer_fwd(desc, flat, x[sl], yj, m, save, scratch)
        C.cephalo_layer_bwd(desc, flat, x[sl], dy[sl], dxj, m, save, Gm, 0.5, j > 0, scratch)
        assert torch.equal(yj, y[sl]) and torch.equal(dxj, dx[sl]), j
    # the gradient: the same fp32 products, the micro-batches added in the accumulators instead of one after the other
    assert float((G - Gm).norm() / Gm.norm()) <= 1e-5


@pytest.mark.parametrize("kind,dtype", [("gpt", "bf16"), ("llama", "bf16"), ("gpt", "f32"), ("llama", "f32")])
@pytest.mark.parametrize("S,m,l", [(512, 3, 12), (509, 3, 11), (512, 2, 9)])             # (more than 16384 tokens: both streams; odd counts; 9216 tokens that the pool does not take at once)
def test_two_streams_take_a_large_share_to_the_same_bits(S, m, l, kind, dtype):
    print(S, m, l, kind, dtype, flush=True)
    desc = C.layer_desc(64, 1, 256, S, True, C.F32 if dtype == "f32" else C.BF16, 1e-5, C.LAYER_LLAMA if kind == "llama" else C.LAYER_GPT)
    assert C.cephalo_share_runs(desc, m * l, m, True)[0] == 2 and C.cephalo_share_runs(desc, m * l, m, False)[0] == 1
    one, two = _share(desc, m * l, m), _share(desc, m * l, m, side=True)
    assert all(torch.equal(a, b) for a, b in zip(one, two))


@pytest.mark.parametrize("kind,dtype", [(C.LAYER_GPT, C.BF16), (C.LAYER_LLAMA, C.BF16), (C.LAYER_GPT, C.F32)], ids=["gpt", "llama", "gpt_f32"])
@pytest.mark.parametrize("S,m,l,V,streams", [(37, 1, 5, 77, 1), (512, 3, 12, 1031, 2), (64, 2, 4, 30011, 1)])      # (small logits; two streams; one micro-batch of logits at a time)
def test_stack_forms_agree_bit_for_bit(kind, dtype, S, m, l, V, streams):
    print(kind, dtype, S, m, l, V, flush=True)
    layer = C.layer_desc(64, 2, 256, S, True, dtype, 1e-5, kind)
    g = torch.Generator(device="cuda").manual_seed(3)
    ids, tgt = (torch.randint(0, V, (m * l, S), device="cuda", generator=g, dtype=torch.int32) for _ in range(2))
    got = []
    for checkpoint, interleave, mb in ((0, 0, m), (0, 1, m), (1, 0, m), (1, 1, m), (0, 0, m * l)):
        sd = C.StackDesc(layer, 2, V, checkpoint, 0, interleave)
        assert C.cephalo_stack_runs(sd, m * l, mb)[0] == (streams if interleave else 1)
        flat = _flat(C.cephalo_stack_param_count(sd), dtype)
        G, loss = torch.full((flat.numel(),), float("nan"), device="cuda"), torch.full((1,), float("nan"), device="cuda")
        ws = _bytes(C.cephalo_stack_workspace_bytes(sd, m * l, mb))
        if interleave:
            C.cephalo_stack_step_interleaved(sd, flat, ids, tgt, m * l, mb, G, 1.0, loss, ws, torch.cuda.Stream())
        else:
            C.cephalo_stack_step(sd, flat, ids, tgt, m * l, mb, G, 1.0, loss, ws)
        torch.cuda.synchronize()
        assert not torch.isnan(G).any()
        got.append((loss, G))
    for loss, G in got[1:4]:
        assert torch.equal(loss, got[0][0]) and torch.equal(G, got[0][1])
    # one micro-batch instead of l: the norms' partial sums differ where a micro-batch is no multiple of 8 rows, in the order of fp32 additions
    assert torch.equal(got[4][0], got[0][0]) and float((got[4][1] - got[0][1]).norm() / got[0][1].norm()) <= 1e-5


@pytest.mark.parametrize("S,m,l,hidden", [(1, 1, 1, 64), (31, 1, 1, 72), (33, 1, 2, 264), (64, 2, 3, 512)])      # (rows around the 32 of a chunk, columns around the 256 of a block)
def test_bias_gradient_is_the_column_sum_of_dy(S, m, l, hidden):
    """The launch that transposes the weights also copies dy and sums its columns."""
    print(S, m, l, hidden, flush=True)
    desc = C.layer_desc(hidden, hidden // 8, 4 * hidden, S, True, C.BF16, 1e-5, C.LAYER_GPT)
    _, _, dy, _, _, G = _share(desc, m * l, m)
    rows, got = dy.reshape(-1, hidden).double(), G[-hidden:].double()        # (the last tensor: the second feed-forward projection's bias)
    bound = rows.shape[0] * 2.0 ** -24 * rows.abs().sum(0) * 0.5             # one rounding of at most the sum of magnitudes per addition
    assert bool(((got - 0.5 * rows.sum(0)).abs() <= bound).all())


@pytest.mark.parametrize("kind", [C.LAYER_GPT, C.LAYER_LLAMA], ids=["gpt", "llama"])
@pytest.mark.parametrize("S,hidden", [(31, 72), (200, 264)])
def test_column_sums_of_dy_only_where_there_is_a_bias(kind, S, hidden):
    """The partial sums are the scratch area's last region.  A layer without biases leaves it alone."""
    print(kind, S, hidden, flush=True)
    desc = C.layer_desc(hidden, hidden // 8, 4 * hidden, S, True, C.BF16, 1e-5, kind)
    g = torch.Generator(device="cuda").manual_seed(7)
    x, dy = (torch.randn(1, S, hidden, device="cuda", generator=g) for _ in range(2))
    flat, y, dx = _flat(C.cephalo_layer_param_count(desc), desc.dtype), torch.empty_like(x), torch.empty_like(x)
    save, scratch = (_bytes(n) for n in C.cephalo_layer_workspace_bytes(desc, 1))
    C.cephalo_layer_fwd(desc, flat, x, y, 1, save, scratch)
    C.cephalo_layer_bwd(desc, flat, x, dy, dx, 1, save, torch.empty(flat.numel(), device="cuda"), 1.0, False, scratch)
    widest = (8 if kind == C.LAYER_LLAMA else 4) * hidden                 # of 3 * hidden and the feed-forward's first outputs
    region = scratch[-((S + 63) // 64 * widest * 4 + 255) // 256 * 256:]
    assert bool((region == 255).all()) == (kind == C.LAYER_LLAMA)
