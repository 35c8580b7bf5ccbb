"""The grid-wide selection on both sides of its chunk-count rule (2048 chunks of
4096 scores: up to there the emission sums the earlier chunks' counts itself), at
partial chunks, and where a histogram workgroup takes several ragged rounds of
keys, with many ties at the boundary key: bit-exact."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5 * 4096, 5 * 4096 + 1, 2048 * 4096, 2048 * 4096 + 1, (1 << 24) + 4099])
@pytest.mark.parametrize("levels", [0, 3])
def test_select_grid_chunk_rule(gpu, n, levels):
    s = np.random.default_rng(n + levels).random(n, dtype=np.float32)
    if levels:
        s = np.floor(s * levels).astype(np.float32)
    k = int(0.4 * n)
    idx = torch.full((k + 8,), -7, dtype=torch.int32, device="cuda")
    gpu.avits_select(torch.from_numpy(s).cuda(), k, idx[:k])
    got = idx.cpu().numpy()
    np.testing.assert_array_equal(got[:k], oracle.select_topk(s, k))
    assert np.all(got[k:] == -7)
