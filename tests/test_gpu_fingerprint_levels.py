"""Fingerprint trees whose inner levels lie at the edges of their kernels: one block of 64 nodes
more or less, last nodes of one, an odd and sixteen digests, and both sides of the level size up
to which two waves share a node."""
import numpy as np
import pytest
import torch

import paper_2608_06690_amd as P
from oracle import pmpe_oracle as O

pytestmark = pytest.mark.gpu

KIB = 1024


@pytest.mark.parametrize("leaves", [2, 15, 16, 18, 63 * 16, 64 * 16, 64 * 16 + 1, 64 * 16 + 3, 65 * 16, 130 * 16 + 7,
                                    32768 * 16, 32768 * 16 + 1])
def test_inner_levels(leaves):
    n = leaves * KIB - 5
    rng = np.random.default_rng(leaves)
    block = rng.integers(0, 256, min(n, 1 << 22), dtype=np.uint8)
    data = np.resize(block, n)
    data[:: 1 << 20] += np.arange(len(data[:: 1 << 20]), dtype=np.uint8)  # no two leaves' parents alike
    dig = torch.empty(32, dtype=torch.uint8, device="cuda")
    ws = torch.empty(P.pmpe_fingerprint_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    P.pmpe_fingerprint(torch.from_numpy(data).cuda(), dig, ws)
    assert bytes(dig.cpu().numpy()) == O.fingerprint(data.tobytes())
