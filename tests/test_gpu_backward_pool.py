"""The router part of the pool-softmax backward at its edges: token counts around the one or four
tokens of a dx block, private pools around the 16 experts of a router-gradient block, hidden sizes
that leave part of a block idle, and both router kernels behind the recomputed logits, or none."""
import pytest
import torch

import paper_2608_06690_amd as P
from tests import pmpe_cases as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,hidden,n_pub,n_priv,k", [
    (1, 128, 5, 4, 2), (7, 384, 20, 16, 3), (66, 640, 16, 17, 2), (130, 256, 70, 33, 4),
    (2049, 256, 24, 8, 2),    # H split, partial logits in the row-gradient buffer
    (2100, 128, 256, 20, 1),  # the partial logits would not fit it: one piece
    (2049, 256, 70, 8, 2),    # H split by the router kernel (fewer logits are recomputed where they are used)
    (1024, 2048, 8, 8, 2), (1025, 2048, 8, 8, 2),  # logits inside and one token to a dx block; the router kernel and four
    (1025, 2176, 7, 6, 2),    # logits inside, four tokens to a block, one in the last
    (2051, 1152, 16, 8, 2),   # the router kernel, four tokens to a block, three in the last
])
@pytest.mark.parametrize("transposed", [True, False])
def test_pool_softmax_router_gradients(tokens, hidden, n_pub, n_priv, k, transposed):
    inter, E = 128, n_pub + n_priv
    d = P.make_desc(hidden, inter, n_pub, n_priv, k, gate_mode=P.PMPE_GATE_POOL_SOFTMAX)
    g = torch.Generator(device="cuda").manual_seed(tokens + hidden)

    def rand(*shape, std=1.0, dtype=torch.bfloat16):
        return torch.empty(*shape, dtype=dtype, device="cuda").normal_(0, std, generator=g)

    wr, bias = rand(E, hidden, std=hidden ** -0.5, dtype=torch.float32), rand(E, dtype=torch.float32)
    w13, w2 = rand(E, 2 * inter, hidden, std=hidden ** -0.5), rand(E, hidden, inter, std=inter ** -0.5)
    layer = P.PolicyMaskedMoE(d, wr[:n_pub], wr[n_pub:], bias, w13[:n_pub], w2[:n_pub], w13[n_pub:], w2[n_pub:])
    x, dout = rand(tokens, hidden), rand(tokens, hidden)
    allow = torch.rand(tokens, generator=g, device="cuda") < 0.5
    words = torch.where(allow, torch.tensor(P.PMPE_POLICY_ALLOW - 2**32, device="cuda"), 0).to(torch.int32)
    b = layer.forward(x, words, layer.audit_buffers(tokens, 1), train=True)
    got = layer.backward(x, dout, b, transposed=transposed)

    idx = b.topk_idx.reshape(tokens, k).long()
    xd, go = x.double(), dout.double()
    z = xd @ wr.double().t() + bias.double()
    pool = torch.zeros(tokens, E, dtype=torch.bool, device="cuda")
    pool[:, :n_pub], pool[:, n_pub:] = ~allow[:, None], allow[:, None]
    p = torch.softmax(z.masked_fill(~pool, float("-inf")), dim=1)
    gate, dg, dx = p.gather(1, idx), torch.zeros(tokens, k, dtype=torch.float64, device="cuda"), torch.zeros_like(xd)
    for e in range(E):
        rows, slot = (idx == e).nonzero(as_tuple=True)
        if rows.numel() == 0:
            continue
        ab = xd[rows] @ w13[e].double().t()
        a, u = ab[:, :inter], ab[:, inter:]
        s = torch.sigmoid(a)
        dg[rows, slot] = (go[rows] * ((a * s * u) @ w2[e].double().t())).sum(1)
        dh = gate[rows, slot][:, None] * go[rows] @ w2[e].double()
        dx.index_add_(0, rows, torch.cat([dh * u * s * (1 + a * (1 - s)), dh * a * s], 1) @ w13[e].double())
    up = torch.zeros_like(z).scatter_(1, idx, dg)
    dz = p * (up - (gate * dg).sum(1, keepdim=True))
    dx += dz @ wr.double()
    # bf16 y, dh and [da; db] as in the other backward tests
    assert C.rel_l2(got.dx.cpu().double().numpy(), dx.cpu().numpy()) <= C.RTOL_BF16
    want = (dz.t() @ xd)[n_pub:]
    assert C.rel_l2(got.dwr_priv.cpu().double().numpy(), want.cpu().numpy()) <= C.RTOL_BF16
    assert got.grad_rows.tolist() == [int((idx == n_pub + e).sum()) for e in range(n_priv)]
