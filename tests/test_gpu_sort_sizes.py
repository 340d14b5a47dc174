"""The radix sort at the tile counts where its passes change form: one group
of tiles, the first with two, the last whose tiles add up their own offsets
and the first whose counts are scanned; keys and order against a stable sort."""
import numpy as np
import pytest

import scenegen as sg
from oracle import build_ref as br

pytestmark = pytest.mark.gpu

TILE, GROUP, DIRECT = 2048, 16, 1024


@pytest.mark.parametrize("n", [4097, TILE * GROUP, TILE * GROUP + 1, 2 * TILE * GROUP + 77, TILE * DIRECT,
                               TILE * DIRECT + 1])
@pytest.mark.parametrize("equal", [False, True])
def test_sorted_keys_and_order(n, equal):
    import torch
    import paper_2001_09792_amd as rg
    rng = np.random.default_rng(n)
    c = rng.uniform(-1.0, 1.0, (n, 1, 3)).astype(np.float32)
    if equal:   # a few hundred distinct keys: long runs whose order is the input's
        c = np.round(c * 4.0) / 4.0
    tri = np.array([[0.0, 0.0, 0.0], [0.01, 0.0, 0.0], [0.0, 0.01, 0.0]], np.float32)
    verts = (c + tri).astype(np.float32).reshape(-1, 3)
    idx = np.arange(3 * n, dtype=np.uint32).reshape(n, 3)
    print(f"[sort] n={n} equal={equal}", flush=True)
    st = rg.lbvh_stages(torch.from_numpy(verts).cuda(), torch.from_numpy(idx.view(np.int32)).cuda())
    keys, ids = br.sort_pairs(br.morton_keys(verts, idx))
    assert np.array_equal(st["keys"].cpu().numpy().view(np.uint64), keys)
    assert np.array_equal(st["ids"].cpu().numpy().view(np.uint32), ids)
