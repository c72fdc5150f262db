"""pmpe_audit alone: request sums, total and violations against numpy, with one lane and with
one wave per request, with ragged and empty requests."""
import numpy as np
import pytest
import torch

import paper_2608_06690_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,requests", [(1, 1), (63, 2), (65, 64), (1111, 37), (256, 256), (200, 300), (1025, 1),
                                             (16385, 32), (68, 17), (69, 17), (64, 16), (4096, 256), (4097, 256), (40000, 5000), (70, 0)])
def test_audit_sums(tokens, requests):
    rng = np.random.default_rng([tokens, requests])
    # counts up to 2^31 (sums need 64 bits), mostly zero under deny, some violations
    rows = rng.integers(0, 2**31, tokens).astype(np.int64) * (rng.random(tokens) < 0.6)
    allow = (rng.random(tokens) < 0.7).astype(np.uint8)
    cuts = np.sort(rng.integers(0, tokens + 1, max(requests - 1, 0)))  # repeated cuts: empty requests
    off = np.concatenate([[0], cuts, [tokens]]).astype(np.int32)
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
