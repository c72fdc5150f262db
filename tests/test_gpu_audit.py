"""pmpe_audit alone: request sums, total and violations against numpy, with one lane and with
one wave per request, with ragged and empty requests, long ones among short ones included."""
import numpy as np
import pytest
import torch

import paper_2608_06690_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,requests", [(1, 1), (63, 2), (65, 64), (1111, 37), (256, 256), (200, 300), (1025, 1),
                                             (16385, 32), (68, 17), (69, 17), (64, 16), (4096, 256), (4097, 256), (40000, 5000), (70, 0)])
def test_audit_sums(tokens, requests):
    rng = np.random.default_rng([tokens, requests])

    def cut():  # repeated cuts: empty requests
        cuts = np.sort(rng.integers(0, tokens + 1, max(requests - 1, 0)))
        return np.concatenate([[0], cuts, [tokens]]).astype(np.int32)

    check(rng, tokens, requests, cut)


def check(rng, tokens, requests, offsets):
    # counts up to 2^31 (sums need 64 bits), mostly zero under deny, some violations
    rows = rng.integers(0, 2**31, tokens).astype(np.int64) * (rng.random(tokens) < 0.6)
    allow = (rng.random(tokens) < 0.7).astype(np.uint8)
    off = offsets()
    d = P.make_desc(128, 64, 2, 2, 1)
    dev = lambda v, dt: torch.from_numpy(np.ascontiguousarray(v)).to(dt).cuda()  # noqa: E731
    out = torch.full((max(requests, 1),), -1, dtype=torch.int64, device="cuda")
    total = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    viol = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    P.pmpe_audit(d, tokens, dev(rows, torch.int32), dev(allow, torch.uint8),
                 dev(off, torch.int32) if requests else None, requests, out if requests else None, total, viol)
    if requests == 0:
        assert int(total) == 0 and int(viol) == 0
        return
    want = [int(rows[off[r]:off[r + 1]].sum()) for r in range(requests)]
    assert out.tolist() == want
    assert int(total) == sum(want)
    assert int(viol) == int(((allow == 0) & (rows > 0)).sum())


# lengths of the requests around the limits of a lane (16 and 64 tokens) and of a wave's rounds (64, 256,
# 512): long requests first, last and among one-token and empty ones, so many of 17 to 64 tokens that
# the limit goes up, more requests than threads
MIXES = [[1] * 200 + [500], [500] + [1] * 200, [16, 17, 63, 64, 65, 256, 257, 512, 513, 4096] + [1] * 60,
         [0, 17] * 400, [40] * 300 + [1] * 900, [65] * 130 + [0] * 5, [3000] * 70, [1] * 2000 + [600] * 40 + [2] * 500,
         [5] * 16, [30] * 64, [4] * 64]


@pytest.mark.parametrize("lengths", MIXES, ids=range(len(MIXES)))
def test_long_requests_among_short_ones(lengths):
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    check(np.random.default_rng(len(lengths)), int(off[-1]), len(lengths), lambda: off)


def test_one_long_request_does_not_hold_up_the_short_ones():
    """200 requests of one token and one of 500 take a few times as long as 200 of 3 or 4 tokens (about
    1.5 times; walked by one lane, the long one made it 13)."""
    d = P.make_desc(128, 64, 2, 2, 1)
    tokens, requests = 700, 201
    rows = torch.ones(tokens, dtype=torch.int32, device="cuda")
    allow = torch.ones(tokens, dtype=torch.uint8, device="cuda")
    out = torch.empty(requests, dtype=torch.int64, device="cuda")
    total, viol = torch.empty(1, dtype=torch.int64, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")

    def microseconds(off):
        off = torch.tensor(off, dtype=torch.int32, device="cuda")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(50):
                P.pmpe_audit(d, tokens, rows, allow, off, requests, out, total, viol)
        best = float("inf")
        for _ in range(5):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            graph.replay()
            t[1].record()
            torch.cuda.synchronize()
            best = min(best, t[0].elapsed_time(t[1]) / 50 * 1e3)
        return best

    even = microseconds([tokens * r // requests for r in range(requests + 1)])
    skewed = microseconds(list(range(201)) + [tokens])
    assert skewed < 5 * even, (skewed, even)
