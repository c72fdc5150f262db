"""The 256 x 256 grouped GEMM (batches of many rows per expert on average) at the edges
of its tiles: row counts around 128 and 256, K loops of one to a few steps, output widths that
are not multiples of a tile, gathered and permuted rows, the shared group, saved projections."""
import numpy as np
import pytest
import torch

import paper_2608_06690_amd as P
from paper_2608_06690_amd import _native as N
from tests import pmpe_cases as C

pytestmark = pytest.mark.gpu

COUNTS = [
    [127, 129, 0, 256, 257, 1],       # both sides of a half tile and of a tile, an empty expert
    [128, 385, 64, 511, 2, 130],
    [0, 0, 0, 1537, 0, 3],            # one expert with many M tiles (more than one chunk of them)
    [159, 160, 161, 191, 192, 193],   # row blocks of a second half that hold valid rows
    [145, 224, 225, 416, 417, 449],   # the same in a second M tile
    [63, 64, 65, 319, 320, 321],      # few row blocks in a first half
]
SHAPES = [(128, 64), (384, 192), (1664, 320)]  # (hidden, inter)


def reference(x, rows, w13, w2, width):
    """fp32 products on the bf16 operands, h and y rounded as the kernel rounds them."""
    ab = x[rows].float() @ w13.float().t()
    h = (torch.nn.functional.silu(ab[:, :width]) * ab[:, width:]).bfloat16().float()
    return ab, (h @ w2.float().t()).bfloat16()


@pytest.mark.parametrize("counts", COUNTS, ids=["edges", "mixed", "tall", "blocks", "second", "short"])
@pytest.mark.parametrize("hidden,inter", SHAPES)
@pytest.mark.parametrize("form", ["gather", "permuted", "train", "shared"])
def test_tile_edges(counts, hidden, inter, form):
    n = 3
    T = sum(counts)
    assert T >= 128 * 2 * n  # the 256 x 256 kernel runs
    shared = form == "shared"
    d = P.make_desc(hidden, inter, n, n, 1, 1 if shared else 0, inter if shared else 0)
    g = torch.Generator(device="cuda").manual_seed(hidden + inter + T)

    def rand(*shape, std=1.0):
        return torch.empty(*shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)

    std = hidden ** -0.5
    x = rand(T, hidden)
    w13, w2 = rand(2 * n, 2 * inter, hidden, std=std), rand(2 * n, hidden, inter, std=inter ** -0.5)
    w13s, w2s = (rand(2 * inter, hidden, std=std), rand(hidden, inter, std=inter ** -0.5)) if shared else (None, None)
    row_token = torch.randperm(T, generator=g, device="cuda").to(torch.int32)
    count = torch.tensor(counts, dtype=torch.int32, device="cuda")
    offset = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    x_perm = x[row_token.long()].contiguous() if form == "permuted" else None
    # a guard row before and after the outputs: nothing outside them may be written
    y_all = torch.full((T + 2, hidden), 7.0, dtype=torch.bfloat16, device="cuda")
    ys_all = torch.full((T + 2, hidden), 7.0, dtype=torch.bfloat16, device="cuda") if shared else None
    ab_all = torch.full((T + 2, 2 * inter), 7.0, device="cuda") if form == "train" else None
    y, ys, ab = (None if t is None else t[1:-1] for t in (y_all, ys_all, ab_all))
    audit = torch.zeros(T, dtype=torch.int32, device="cuda")
    calls = torch.zeros(n, dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(P.pmpe_workspace_bytes(d, T), dtype=torch.uint8, device="cuda")
    args = (d, T, x_perm, x, count, offset, row_token, w13[:n], w2[:n], w13[n:], w2[n:], w13s, w2s, ys, y, audit,
            calls, status)
    if form == "train":
        P.pmpe_expert_ffn_train(*args, ab, ws)
    else:
        P.pmpe_expert_ffn(*args, ws)
    torch.cuda.synchronize()
    off = offset.tolist()
    for e in range(2 * n):
        if counts[e] == 0:
            continue
        sl = slice(off[e], off[e + 1])
        ab_ref, y_ref = reference(x, row_token[sl].long(), w13[e], w2[e], inter)
        assert C.rel_l2(y[sl].cpu().double().numpy(), y_ref.cpu().double().numpy()) <= C.RTOL_ROW_BF16, e
        if form == "train":
            # fp32 sums of up to 1664 products in another order: about sqrt(1664) 2^-24 = 2.4e-6
            assert C.rel_l2(ab[sl].cpu().double().numpy(), ab_ref.cpu().double().numpy()) <= 1e-5, e
    if shared:
        _, y_ref = reference(x, torch.arange(T, device="cuda"), w13s, w2s, inter)
        assert C.rel_l2(ys.cpu().double().numpy(), y_ref.cpu().double().numpy()) <= C.RTOL_ROW_BF16
    for t in (y_all, ys_all, ab_all):
        if t is not None:
            assert bool((t[0] == 7).all()) and bool((t[-1] == 7).all())
    want = torch.zeros(T, dtype=torch.int32, device="cuda")
    want[row_token[off[n]:].long()] = 1
    assert torch.equal(audit, want)
    assert calls.tolist() == [int(c > 0) for c in counts[n:]]
    assert int(status) == 0


# the last batch of the 64-row tiles and the first of the 256-row ones, for hidden sizes that make at
# least four, two and less than two 256 x 256 tiles per CU with 64 experts
@pytest.mark.parametrize("hidden,tokens", [(4096, 52 * 64 - 1), (4096, 52 * 64), (2048, 64 * 64 - 1), (2048, 64 * 64),
                                           (1024, 128 * 64 - 1), (1024, 128 * 64)])
def test_both_sides_of_the_tile_choice(hidden, tokens):
    n, inter = 32, 64
    d = P.make_desc(hidden, inter, n, n, 1)
    g = torch.Generator(device="cuda").manual_seed(tokens)
    x = torch.empty(tokens, hidden, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    w13 = torch.empty(2 * n, 2 * inter, hidden, dtype=torch.bfloat16, device="cuda").normal_(0, hidden ** -0.5, generator=g)
    w2 = torch.empty(2 * n, hidden, inter, dtype=torch.bfloat16, device="cuda").normal_(0, inter ** -0.5, generator=g)
    expert = torch.sort(torch.randint(0, 2 * n, (tokens,), generator=g, device="cuda")).values
    count = torch.bincount(expert, minlength=2 * n).to(torch.int32)
    offset = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), count.cumsum(0)]).to(torch.int32)
    row_token = torch.randperm(tokens, generator=g, device="cuda").to(torch.int32)
    y = torch.empty(tokens, hidden, dtype=torch.bfloat16, device="cuda")
    audit = torch.zeros(tokens, dtype=torch.int32, device="cuda")
    ws = torch.empty(P.pmpe_workspace_bytes(d, tokens), dtype=torch.uint8, device="cuda")
    P.pmpe_expert_ffn(d, tokens, None, x, count, offset, row_token, w13[:n], w2[:n], w13[n:], w2[n:], None, None, None,
                      y, audit, None, None, ws)
    for e in range(2 * n):
        sl = slice(int(offset[e]), int(offset[e + 1]))
        _, y_ref = reference(x, row_token[sl].long(), w13[e], w2[e], inter)
        assert C.rel_l2(y[sl].cpu().double().numpy(), y_ref.cpu().double().numpy()) <= C.RTOL_ROW_BF16, e
    assert int(audit.sum()) == int(count[n:].sum())


# Several tiles per block, in rows of every kind (none, part of one half, one half, both, several M tiles): the
# copies of a tile are then in flight while the one or two before it still multiply and store. K = 64 makes
# one step per tile (GEMM2 of 4096 x 64, more than five tiles per block), 128 two (GEMM1 of 128 x 2048). The
# last shape gives a block more tiles than the 256 whose descriptions it keeps.
@pytest.mark.parametrize("hidden,inter,n", [(4096, 64, 48), (128, 2048, 48), (128, 65536, 80)])
def test_many_tiles_per_block(hidden, inter, n):
    rng = np.random.default_rng(inter)
    kinds = [lambda: 0, lambda: rng.integers(1, 65), lambda: 128, lambda: rng.integers(129, 193), lambda: 256,
             lambda: rng.integers(193, 300)]
    counts = [int(kinds[rng.integers(6)]()) for _ in range(2 * n)]
    counts[-1] = max(1, 128 * 2 * n - sum(counts[:-1]))  # the 256 x 256 kernel runs
    T = sum(counts)
    blocks = 256
    tiles = sum((c + 255) // 256 for c in counts) * max((inter + 127) // 128, (hidden + 255) // 256)
    assert tiles > (256 if inter == 65536 else 5) * blocks
    d = P.make_desc(hidden, inter, n, n, 1)
    g = torch.Generator(device="cuda").manual_seed(inter)
    x = torch.empty(T, hidden, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    w13 = torch.empty(2 * n, 2 * inter, hidden, dtype=torch.bfloat16, device="cuda").normal_(0, hidden ** -0.5, generator=g)
    w2 = torch.empty(2 * n, hidden, inter, dtype=torch.bfloat16, device="cuda").normal_(0, inter ** -0.5, generator=g)
    offset = np.concatenate([[0], np.cumsum(counts)])
    count = torch.tensor(counts, dtype=torch.int32, device="cuda")
    off = torch.tensor(offset, dtype=torch.int32, device="cuda")
    row_token = torch.randperm(T, generator=g, device="cuda").to(torch.int32)
    ws = torch.empty(P.pmpe_workspace_bytes(d, T), dtype=torch.uint8, device="cuda")
    for priv in (True, False):  # private weights given, and missing
        y = torch.full((T, hidden), 7.0, dtype=torch.bfloat16, device="cuda")
        audit = torch.zeros(T, dtype=torch.int32, device="cuda")
        calls = torch.zeros(n, dtype=torch.int32, device="cuda")
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        P.pmpe_expert_ffn(d, T, None, x, count, off, row_token, w13[:n], w2[:n], w13[n:] if priv else None,
                          w2[n:] if priv else None, None, None, None, y, audit, calls, status, ws)
        torch.cuda.synchronize()
        for e in range(2 * n):
            if counts[e] == 0:
                continue
            sl = slice(offset[e], offset[e + 1])
            if e >= n and not priv:
                assert not bool(y[sl].any()), e
                continue
            _, y_ref = reference(x, row_token[sl].long(), w13[e], w2[e], inter)
            # row by row: a single wrong tile may not hide in the norm of the others
            err = (y[sl].float() - y_ref.float()).norm(dim=1) / y_ref.float().norm(dim=1)
            assert float(err.max()) <= C.RTOL_ROW_BF16, (e, int(err.argmax()))
        want = torch.zeros(T, dtype=torch.int32, device="cuda")
        if priv:
            want[row_token[offset[n]:].long()] = 1
        assert torch.equal(audit, want)
        assert calls.tolist() == [int(c > 0 and priv) for c in counts[n:]]
        assert int(status) == (0 if priv else N.PMPE_DEV_PRIV_WEIGHTS_MISSING)
