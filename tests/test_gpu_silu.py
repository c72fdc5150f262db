"""h = silu(g) u of the bf16 paths is the fp32 value rounded once: the same bits as the fp32 layer's h
rounded to bf16, whatever the path (tiles of 64 and of 256 rows, saved projections, fp8 weights,
the LoRA arm).

The layer's weights pick columns of x, so that its output is h itself: g is the sum of one x value and
2^-8 of another (both multiples of 1/16 below 8: exact in any order of summation), u a third
one, and W2 the identity. Of 16.8 million values about one in 25 changes by an ulp of fp32 when the
division of silu becomes a product with a 1-ulp reciprocal, and one in 65536 of those lies at
a rounding boundary of bf16."""
import pytest
import torch

import paper_2608_06690_amd as P

pytestmark = pytest.mark.gpu

H = I = 512
T = 32767  # a ragged last tile


def weights(n, dtype, one, eps):
    """w13 [n, 2I, H] and w2 [n, H, I] of `dtype` whose values 1 and 2^-8 are spelled one and eps."""
    i = torch.arange(I, device="cuda")
    w13 = torch.zeros(2 * I, H, dtype=dtype, device="cuda")
    w13[i, i] = one
    w13[i, (i + 3) % H] = eps
    w13[I + i, (i + 1) % H] = one
    w2 = torch.zeros(H, I, dtype=dtype, device="cuda")
    w2[i, i] = one
    return w13.expand(n, -1, -1).contiguous(), w2.expand(n, -1, -1).contiguous()


def inputs():
    g = torch.Generator(device="cuda").manual_seed(11)
    return torch.randint(-127, 128, (T, H), generator=g, device="cuda").float() / 16


def run(form, x):
    # experts per pool: 128 take at most 128 rows each (64-row tiles), one takes them all (256)
    n = 1 if form in ("f32", "bf16_256", "train_256", "fp8_256") else 128
    f32 = form == "f32"
    d = P.make_desc(H, I, n, n, 1, bf16=not f32)
    x = x if f32 else x.bfloat16()
    if form.startswith("fp8"):
        w13, w2 = weights(2 * n, torch.uint8, 0x38, 0x02)  # e4m3 1 and 2^-8
    else:
        w13, w2 = weights(2 * n, x.dtype, 1.0, 2.0 ** -8)
    count = torch.full((2 * n,), T // (2 * n), dtype=torch.int32, device="cuda")
    count[0] += T - int(count.sum())
    if form == "lora":  # public experts only
        count[:n] += count[n:]
        count[n:] = 0
    offset = torch.zeros(2 * n + 1, dtype=torch.int32, device="cuda")
    offset[1:] = count.cumsum(0)
    rows = torch.arange(T, dtype=torch.int32, device="cuda")
    y = torch.empty(T, H, dtype=x.dtype, device="cuda")
    audit = torch.zeros(T, dtype=torch.int32, device="cuda")
    ws = torch.empty(P.pmpe_workspace_bytes(d, T), dtype=torch.uint8, device="cuda")
    pools = (w13[:n], w2[:n], w13[n:], w2[n:])
    if form.startswith("fp8"):
        d.w_dtype = P.PMPE_FP8_E4M3
        s13, s2 = torch.ones(2 * n, 2 * I, device="cuda"), torch.ones(2 * n, H, device="cuda")
        P.pmpe_expert_ffn_fp8(d, T, None, x, count, offset, rows, *pools, s13[:n], s2[:n], s13[n:], s2[n:], y, audit,
                              None, None, ws)
    elif form.startswith("train"):
        ab = torch.empty(T, 2 * I, device="cuda")
        P.pmpe_expert_ffn_train(d, T, None, x, count, offset, rows, *pools, None, None, None, y, audit, None, None, ab, ws)
    elif form == "lora":  # adapters that add nothing
        R = 8
        z = lambda *s: torch.zeros(n, *s, dtype=x.dtype, device="cuda")  # noqa: E731
        words = torch.full((T,), P.PMPE_POLICY_ALLOW - 2**32, dtype=torch.int64, device="cuda").to(torch.int32)
        ws = torch.empty(P.pmpe_expert_ffn_lora_workspace_bytes(d, T), dtype=torch.uint8, device="cuda")
        P.pmpe_expert_ffn_lora(d, T, None, x, count, offset, rows, words, *pools[:2], z(2 * R, H), z(I, R), z(I, R),
                               z(R, I), z(H, R), R, 1.0, P.PMPE_LORA_GATE_ROW, y, audit, None, ws)
    else:
        P.pmpe_expert_ffn(d, T, None, x, count, offset, rows, *pools, None, None, None, y, audit, None, None, ws)
    return y


@pytest.mark.parametrize("form", ["bf16_64", "bf16_256", "train_64", "train_256", "fp8_64", "fp8_256", "lora"])
def test_h_is_the_rounded_fp32_value(form):
    x = inputs()
    want = run("f32", x).bfloat16()
    got = run(form, x)
    assert float(want.float().abs().max()) > 8
    assert int((got != want).sum()) == 0


def test_silu_of_extreme_projections():
    """Waves with |g| of 87 and more divide: the same bits as the fp32 layer's, down to g / inf = -0."""
    x = torch.zeros(T, H, device="cuda")
    g = torch.tensor([-3e38, -1e30, -1000.0, -200.0, -89.0, -88.5, -88.0, -87.5, -87.0, -86.0, 86.0, 87.0, 88.0, 1e30,
                      3e38, -0.0], device="cuda").bfloat16().float()
    # columns 0, 8, 16, ... are the g of elements i = 0 mod 8; their u columns are 1
    x[:, 0::8] = g.repeat(4)[None, :]
    x[:, 1::8] = 1.0
    want = run("f32", x).bfloat16()[:, 0::8]
    assert bool(want.isfinite().all())
    for form in ("bf16_64", "bf16_256"):
        assert torch.equal(run(form, x)[:, 0::8].contiguous().view(torch.int16), want.contiguous().view(torch.int16)), form
