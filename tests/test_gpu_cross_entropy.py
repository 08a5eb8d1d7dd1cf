"""Cross-entropy rows against the definition in 64 bits, at the sizes where the kernel changes its form."""
import pytest
import torch

import paper_2411_01075_amd as C

pytestmark = pytest.mark.gpu

# rows, classes, pitch: a wavefront, 256 and 1024 threads a row at both numbers of groups, the two-pass form, blocks with several rows, one row
SIZES = [(1, 5, 8), (9, 1031, 1088), (5000, 300, 320), (700, 2048, 2048), (300, 8191, 8192), (1100, 8200, 8256), (800, 16380, 16384), (600, 32761, 32768),
         (261, 50257, 50304), (40, 57345, 57408), (300, 65536, 65536), (3, 65537, 65600)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,V,ld", SIZES)
def test_cross_entropy_rows(rows, V, ld, dtype):
    print("cross entropy", rows, V, ld, dtype, flush=True)
    g = torch.Generator(device="cuda").manual_seed(V)
    x = torch.randn(rows, ld, device="cuda", generator=g) * 3
    x[:, V:] = float("nan")                                       # (the padding is not read as a class)
    if ld <= 65536:
        x[0, : V // 2] = float("-inf")                            # half of a row masked, its first groups wholly
    tgt = torch.randint(0, V, (rows,), device="cuda", generator=g, dtype=torch.int32)
    tgt[0] = V - 1
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    d, again = (torch.full((rows, ld), float("nan"), device="cuda", dtype=dt) for _ in range(2))
    loss = torch.full((rows,), float("nan"), device="cuda")
    C.cephalo_op_cross_entropy(C.BF16 if dtype == "bf16" else C.F32, x, ld, tgt, d, loss, rows, V, 0.25)
    C.cephalo_op_cross_entropy(C.BF16 if dtype == "bf16" else C.F32, x, ld, tgt, again, loss, rows, V, 0.25)
    assert torch.equal(d, again) and not d[:, V:].any()
    z = x[:, :V].double()
    lse = torch.logsumexp(z, -1)
    at = torch.arange(rows, device="cuda")
    assert float((loss.double() - (lse - z[at, tgt.long()])).abs().max()) <= 1e-5
    want = torch.exp(z - lse[:, None])
    want[at, tgt.long()] -= 1
    want *= 0.25
    # a probability carries a handful of fp32 roundings and those of an exponent of up to 64 (2^-17 of it), then one rounding to the result's type
    # (half a unit: 2^-9 of a bf16 value); at the target 1 is taken off, which leaves the probability's own error
    err, p = (d[:, :V].double() - want).abs(), torch.exp(z - lse[:, None]) * 0.25
    assert bool((err <= want.abs() * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -22) + p * 2.0 ** -16 + 1e-38).all())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,V,ld", [(9, 1031, 1088), (70, 8191, 8192), (70, 16380, 16384), (261, 50257, 50304), (3, 65537, 65600)])
@pytest.mark.parametrize("offset", [3000.0, -3000.0])
def test_cross_entropy_of_large_logits_and_masks(rows, V, ld, dtype, offset):
    """The result depends on differences of logits only, however large they are; a mask may be the type's lowest value."""
    print("cross entropy", rows, V, ld, dtype, offset, flush=True)
    g = torch.Generator(device="cuda").manual_seed(V)
    x = torch.randn(rows, ld, device="cuda", generator=g) * 3 + offset
    lowest = torch.finfo(torch.float32).min
    x[0, : V // 2] = lowest                                       # half of a row, its first groups wholly; every other column; every column but one
    x[1, ::2] = lowest
    x[2, : V - 1] = lowest
    tgt = torch.randint(V // 2, V, (rows,), device="cuda", generator=g, dtype=torch.int32)
    tgt[1], tgt[2] = V // 2 * 2 - 1, V - 1
    d = torch.full((rows, ld), float("nan"), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    loss = torch.full((rows,), float("nan"), device="cuda")
    C.cephalo_op_cross_entropy(C.BF16 if dtype == "bf16" else C.F32, x, ld, tgt, d, loss, rows, V, 0.25)
    z = x[:, :V].double()
    z = z - z.max(-1, keepdim=True).values
    lse = torch.logsumexp(z, -1)
    at = torch.arange(rows, device="cuda")
    # the two-pass form of the widest rows rounds the whole logsumexp: half a unit of 4096
    assert float((loss.double() - (lse - z[at, tgt.long()])).abs().max()) <= (1e-5 if ld <= 65536 else 2.0 ** -12)
    want = torch.exp(z - lse[:, None]) * 0.25
    p = want.clone()
    want[at, tgt.long()] -= 0.25
    # as above; and the two-pass form's rounded logsumexp in every exponent
    err, own = (d[:, :V].double() - want).abs(), 2.0 ** -16 if ld <= 65536 else 2.0 ** -12
    assert bool((err <= want.abs() * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -22) + p * own + 1e-38).all())
