"""Refits on both sides of the rule that puts every level of a small hierarchy
into the one-workgroup launch (480 nodes, at width 8 320, per level past the
levels of up to 256): alone, and together with structures from the other side."""
import numpy as np
import pytest

import scenegen as sg
from tests import bvh_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,leaf,sizes", [
    (2, 1, [400, 1600, 3200, 6400, 30000]),
    (2, 4, [800, 6400, 12800]),
    (4, 1, [300, 1000, 3000, 6400]),
    (4, 4, [3200, 6400, 12800]),
    (8, 1, [300, 800, 3000, 6400]),
    (8, 8, [3200, 20000]),
])
def test_refit_alone_and_together(width, leaf, sizes):
    import torch
    import paper_2001_09792_amd as rg
    meshes = [sg.random_soup(n, 60 + n) for n in sizes] + [sg.torus(28, 28, 1.0, 0.3, 0.05, 5.0, 3)]
    v = [torch.from_numpy(np.ascontiguousarray(m.verts, np.float32)).cuda() for m in meshes]
    i = [torch.from_numpy(np.ascontiguousarray(m.idx, np.uint32).view(np.int32)).cuda() for m in meshes]
    blas = [rg.build_blas(a, b, None, width, leaf) for a, b in zip(v, i)]
    print(f"[refit] W={width} L={leaf}", [(int(b.desc.n_nodes), int(b.desc.depth)) for b in blas], flush=True)
    before = [b.buf.clone() for b in blas]

    def same(b, old):
        d = b.desc
        return torch.equal(b.buf[d.nodes_off: d.slots_off], old[d.nodes_off: d.slots_off])

    moved = [(a * 1.5 + 0.25).contiguous() for a in v]
    for b, a, k, m in zip(blas, moved, i, meshes):
        rg.refit_blas(b, a, k)
        info = bvh_check.check_blas(b.buf.cpu().numpy(), b.desc, refitted=True)
        assert np.array_equal(info["verts"], a.cpu().numpy()[m.idx[info["prim"]]])
    alone = [b.buf.clone() for b in blas]
    rg.refit_blas_many(blas, v, i)
    assert all(same(b, old) for b, old in zip(blas, before))
    rg.refit_blas_many(blas, moved, i)
    assert all(same(b, old) for b, old in zip(blas, alone))
