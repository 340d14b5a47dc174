"""Refits of hierarchies whose levels lie on both sides of the one-workgroup
launch, with leaves of one and of several triangles: new positions give the
boxes that the triangles have, and the old positions give back the build."""
import numpy as np
import pytest

import scenegen as sg
from tests import bvh_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,leaf", [(2, 1), (2, 5), (4, 1), (4, 4), (8, 1), (8, 8)])
@pytest.mark.parametrize("n", [1, 3, 300, 1300, 20000])
def test_refit_boxes_and_back(width, leaf, n):
    import torch
    import paper_2001_09792_amd as rg
    mesh = sg.random_soup(n, 40 + n)
    v = torch.from_numpy(np.ascontiguousarray(mesh.verts, np.float32)).cuda()
    i = torch.from_numpy(np.ascontiguousarray(mesh.idx, np.uint32).view(np.int32)).cuda()
    print(f"[refit] W={width} L={leaf} n={n}", flush=True)
    b = rg.build_blas(v, i, None, width, leaf)
    before = b.buf.clone()
    moved = (v * 1.5 + 0.25).contiguous()
    rg.refit_blas(b, moved, i)
    info = bvh_check.check_blas(b.buf.cpu().numpy(), b.desc, refitted=True)
    assert np.array_equal(info["verts"], moved.cpu().numpy()[mesh.idx[info["prim"]]])
    rg.refit_blas(b, v, i)
    torch.cuda.synchronize()
    d = b.desc
    assert torch.equal(b.buf[d.nodes_off: d.slots_off], before[d.nodes_off: d.slots_off])
