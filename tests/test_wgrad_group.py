"""A layer's weight gradients in one launch: which tile the estimate picks, and each tile's results."""
import dataclasses

import pytest
import torch

import paper_2411_01075_amd as C
from paper_2411_01075_amd import binding


def layer_products(H, F):
    """(out features, in features, has a bias gradient) of a GPT-style layer's projections, in the order in which its backward runs them."""
    return [H, F, H, 3 * H], [F, H, H, H], [0, 1, 0, 1]


def layer_choice(H, F, tokens):
    N, K, bias = layer_products(H, F)
    return binding.cephalo_wgrad_group_tile(tokens, N, K, bias)


# tile, hidden, heads, mlp, tokens a sample, samples a micro-batch, micro-batches: every tile of the group; ragged in every axis
LAYERS = [(0, 800, 10, 3200, 373, 3, 1), (1, 728, 7, 2912, 133, 3, 2), (2, 264, 3, 1032, 61, 4, 2), (3, 640, 8, 2560, 136, 1, 1), (3, 1024, 16, 4096, 73, 1, 1)]


def test_the_layers_below_reach_every_tile():
    for tile, H, _, F, S, m, l in LAYERS:
        assert layer_choice(H, F, S * m * l)[0] == tile, (H, F, S * m * l)
    assert {c[0] for c in LAYERS} == {0, 1, 2, 3}


@pytest.mark.parametrize("H,F,tokens", [(3968, 4784, 4096), (4040, 5080, 1500), (4000, 4872, 2048)])
def test_a_product_with_a_bias_gradient_is_not_priced_at_two_launches(H, F, tokens):
    """With its column sums a weight gradient is one launch.  At these sizes two of them would be faster than the group, one is not."""
    N, K, bias = layer_products(H, F)
    assert binding.cephalo_wgrad_group_tile(tokens, N, K, [0] * 4)[0] == -1
    assert layer_choice(H, F, tokens)[0] == 0


def test_group_entries_refuse_what_they_do_not_take():
    with pytest.raises(binding.CephaloError):
        binding.cephalo_wgrad_group_tile(64, [8] * 5, [8] * 5, [0] * 5)
    with pytest.raises(binding.CephaloError):
        binding.cephalo_wgrad_group_tile(0, [8, 8], [8, 8], [0, 0])
    with pytest.raises(binding.CephaloError):
        binding.cephalo_wgrad_group_tile(64, [8, 12], [8, 8], [0, 0])


@pytest.mark.gpu
@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("T", [1, 63, 200, 1345, 4100])
@pytest.mark.parametrize("N,K", [([8, 136, 72, 264], [72, 8, 264, 8]), ([264, 1032, 520, 776], [1032, 264, 136, 392]), ([520], [392]), ([128, 256], [256, 128])])
def test_group_gives_the_bits_of_single_launches(T, N, K, tile):
    """Every tile adds an output's products in token order; one launch per product does the same unless it cuts the token axis."""
    print("wgrad group", T, N, K, tile, flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + N[0])
    dY = [torch.randn(T, n, device="cuda", generator=g).bfloat16() for n in N]
    X = [torch.randn(T, k, device="cuda", generator=g).bfloat16() for k in K]
    G = [torch.full((n, k), float("nan"), device="cuda") for n, k in zip(N, K)]
    gb = [torch.full((n,), float("nan"), device="cuda") if i % 2 == 1 or len(N) == 1 else None for i, n in enumerate(N)]
    ws = torch.empty(binding.cephalo_op_linear_wgrad_group_workspace(N, K), dtype=torch.uint8, device="cuda").fill_(255)
    binding.cephalo_op_linear_wgrad_group(dY, X, T, N, K, G, gb, 0.5, 0, tile, ws)
    first = [x.clone() for x in G]
    pieces = binding.cephalo_wgrad_group_tile(T, N, K, [0] * len(N))[1]
    eps = 2.0 ** -24
    for i, (n, k) in enumerate(zip(N, K)):
        alone = torch.full((n, k), float("nan"), device="cuda")
        work = torch.empty(C.cephalo_op_linear_wgrad_workspace(C.BF16, T, n, k), dtype=torch.uint8, device="cuda")
        C.cephalo_op_linear_wgrad(C.BF16, dY[i], X[i], T, n, k, alone, 0.5, 0, work)
        if pieces[i] == 1:
            assert torch.equal(G[i], alone), i
        a, b = dY[i].double(), X[i].double()
        ref, size = a.t().contiguous() @ b, a.abs().t().contiguous() @ b.abs()
        assert ((G[i].double() - 0.5 * ref).abs() <= 0.5 * (T + 4) * eps * size).all(), i
        if gb[i] is not None:
            assert ((gb[i].double() - 0.5 * a.sum(0)).abs() <= 0.5 * (T + 12) * eps * a.abs().sum(0)).all(), i
    binding.cephalo_op_linear_wgrad_group(dY, X, T, N, K, G, gb, 1.0, 1, tile, ws)
    for i, (n, k) in enumerate(zip(N, K)):
        once = torch.full((n, k), float("nan"), device="cuda")
        binding.cephalo_op_linear_wgrad_group(dY[i:i + 1], X[i:i + 1], T, [n], [k], [once], [None], 1.0, 0, tile, ws)
        assert torch.equal(G[i], first[i] + once), i


@pytest.mark.gpu
@pytest.mark.parametrize("tile,H,heads,F,S,m,l", LAYERS)
def test_a_layer_on_every_group_tile(tile, H, heads, F, S, m, l):
    from tests import harness as Hn
    from workloads import CONFIGS, draw_activations, draw_layer_params
    assert layer_choice(H, F, S * m * l)[0] == tile
    cfg = dataclasses.replace(CONFIGS["c2"], hidden=H, heads=heads, mlp=F, seq=S, micro_batch=m, n_micro=l)
    tensors = draw_layer_params(cfg, perturbed=True)
    x, dy = draw_activations(cfg)
    Hn.compare_share(cfg, Hn.gpu_share_step(cfg, tensors, x, dy), Hn.oracle_share_step(cfg, tensors, x, dy))
