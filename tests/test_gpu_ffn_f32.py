"""The fp32 expert products at the edges of their row tiles (16 rows with few rows per expert,
64 with more), with uneven K splits, shared experts, gathered and permuted rows."""
import numpy as np
import pytest
import torch

import paper_2608_06690_amd as P
from tests import pmpe_cases as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [[15, 17, 0, 16, 1, 33],       # 16-row tiles
                                    [63, 65, 0, 128, 1, 257]],    # 64-row tiles
                         ids=["small", "large"])
@pytest.mark.parametrize("hidden,inter", [(128, 64), (384, 192)])
@pytest.mark.parametrize("form", ["gather", "permuted", "shared"])
def test_f32_tile_edges(counts, hidden, inter, form):
    n, T, shared = 3, sum(counts), form == "shared"
    d = P.make_desc(hidden, inter, n, n, 1, 1 if shared else 0, inter if shared else 0, bf16=False)
    g = torch.Generator(device="cuda").manual_seed(hidden + T)

    def rand(*shape):
        return torch.randn(*shape, device="cuda", generator=g) * shape[-1] ** -0.5

    x = rand(T, hidden) * hidden ** 0.5
    w13, w2 = rand(2 * n, 2 * inter, hidden), rand(2 * n, hidden, inter)
    w13s, w2s = (rand(2 * inter, hidden), rand(hidden, inter)) if shared else (None, None)
    row_token = torch.randperm(T, generator=g, device="cuda").to(torch.int32)
    off = np.concatenate([[0], np.cumsum(counts)])
    count, offset = (torch.tensor(np.asarray(v), dtype=torch.int32, device="cuda") for v in (counts, off))
    x_perm = x[row_token.long()].contiguous() if form == "permuted" else None
    y_all, ys_all = (torch.full((T + 2, hidden), 7.0, device="cuda") for _ in range(2))
    audit, calls = torch.zeros(T, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    ws = torch.empty(P.pmpe_workspace_bytes(d, T), dtype=torch.uint8, device="cuda")
    P.pmpe_expert_ffn(d, T, x_perm, x, count, offset, row_token, w13[:n], w2[:n], w13[n:], w2[n:], w13s, w2s,
                      ys_all[1:-1] if shared else None, y_all[1:-1], audit, calls, None, ws)

    def ref(rows, a, b):
        ab = x[rows].double() @ a.double().t()
        h = torch.nn.functional.silu(ab[:, :inter]) * ab[:, inter:]
        return (h @ b.double().t()).cpu().numpy()

    for e in range(2 * n):
        if counts[e]:
            sl = slice(off[e], off[e + 1])
            got = y_all[1:-1][sl].cpu().double().numpy()
            assert C.rel_l2(got, ref(row_token[sl].long(), w13[e], w2[e])) <= C.RTOL_ROW_F32, e
    if shared:
        got = ys_all[1:-1].cpu().double().numpy()
        assert C.rel_l2(got, ref(torch.arange(T, device="cuda"), w13s, w2s)) <= C.RTOL_ROW_F32
    for t in (y_all, ys_all):
        assert bool((t[0] == 7).all()) and bool((t[-1] == 7).all())
    want = torch.zeros(T, dtype=torch.int32, device="cuda")
    want[row_token[off[n]:].long()] = 1
    assert torch.equal(audit, want)
    assert calls.tolist() == [int(c > 0) for c in counts[n:]]
