"""Treelet restructuring with one wave per node and the depths near the root
in one launch: hierarchies whose sizes lie around a treelet's leaf count and
around the node count up to which a depth joins that launch, with equal areas
(ties), chains and infinite areas, against the restructuring's definition."""
import numpy as np
import pytest

import scenegen as sg
from oracle import build_ref as br

pytestmark = pytest.mark.gpu


def _mesh(kind, n):
    if kind == "soup":
        return sg.random_soup(n, 100 + n)
    tri = np.array([[0.0, 0.0, 0.0], [0.5, 0.0, 0.25], [0.0, 0.5, 0.0]])
    c = np.zeros((n, 1, 3))
    if kind == "line":      # equal spacing: areas tie
        c[:, 0, 0] = np.arange(n)
    else:                   # "chain": halving distances, one Morton level each
        c[:, 0, 0] = 2.0 ** -np.minimum(np.arange(n), 60)
    return sg.triangles_mesh(c + tri)


@pytest.mark.parametrize("kind", ["soup", "line", "chain"])
@pytest.mark.parametrize("n", [3, 4, 6, 7, 8, 16, 17, 18, 33, 34, 64, 65, 66, 257, 2049])
def test_wave_treelets_match_definition(kind, n):
    import torch
    import paper_2001_09792_amd as rg
    mesh = _mesh(kind, n)
    v = torch.from_numpy(np.ascontiguousarray(mesh.verts, np.float32)).cuda()
    i = torch.from_numpy(np.ascontiguousarray(mesh.idx, np.uint32).view(np.int32)).cuda()
    print(f"[treelet waves] {kind} {n}", flush=True)
    st = rg.lbvh_stages(v, i, builder="treelet", radius=2)
    ref_sorted, ref_ids = br.sort_pairs(br.morton_keys(mesh.verts, mesh.idx))
    lo, hi = br.tri_boxes(mesh.verts, mesh.idx)
    lo, hi = lo[ref_ids], hi[ref_ids]
    left, right, first, last = br.radix_tree(ref_sorted)
    blo, bhi = br.refit(lo, hi, first, last)
    L, R, BLO, BHI = br.treelet_optimise(left, right, lo, hi, blo, bhi, rounds=2)
    rank = br.leaf_order(L, R, n)
    relabel = lambda c: np.where(c < 0, -(rank[np.maximum(-c - 1, 0)] + 1), c).astype(np.int32)
    assert np.array_equal(st["left"].cpu().numpy(), relabel(L))
    assert np.array_equal(st["right"].cpu().numpy(), relabel(R))
    boxes = st["boxes"].cpu().numpy()
    assert np.array_equal(boxes[: n - 1, :3], BLO) and np.array_equal(boxes[: n - 1, 3:], BHI)
