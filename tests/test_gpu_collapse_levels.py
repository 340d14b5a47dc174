"""The wide collapse's levels of bounded size in one workgroup and a queue add
per workgroup above: every hierarchy's wide nodes are well formed at sizes
around the handover (512 nodes of a level), for each width, and the level
table and parents agree with the nodes."""
import numpy as np
import pytest

import scenegen as sg
from tests import bvh_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [2, 4, 8])
@pytest.mark.parametrize("n", [4097, 5000, 8192, 40000])
@pytest.mark.parametrize("builder", ["lbvh", "treelet"])
def test_wide_nodes_level_by_level(width, n, builder):
    import torch
    import paper_2001_09792_amd as rg
    mesh = sg.random_soup(n, 7 * n + width)
    v = torch.from_numpy(np.ascontiguousarray(mesh.verts, np.float32)).cuda()
    i = torch.from_numpy(np.ascontiguousarray(mesh.idx, np.uint32).view(np.int32)).cuda()
    print(f"[collapse] {builder} W={width} n={n}", flush=True)
    b = rg.build_blas(v, i, None, width, 1, builder=builder)
    info = bvh_check.check_blas(b.buf.cpu().numpy(), b.desc)
    assert np.array_equal(info["verts"], mesh.verts[mesh.idx[info["prim"]]])
    d, buf = b.desc, b.buf.cpu().numpy()
    words = buf[d.nodes_off: d.nodes_off + d.n_nodes * 32 * width].view(np.uint32).reshape(d.n_nodes, 8 * width)
    links = words[:, 6 * width: 7 * width]
    # breadth-first numbering: level by level, each node once
    level, seen = np.array([0]), 1
    sizes = [1]
    while True:
        l = links[level]
        nxt = np.sort(l[(l & 0x80000000) == 0])
        if nxt.size == 0:
            break
        assert np.array_equal(nxt, np.arange(seen, seen + nxt.size))
        seen += nxt.size
        sizes.append(nxt.size)
        level = nxt
    assert seen == d.n_nodes
    assert max(sizes) > 512
