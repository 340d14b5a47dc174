"""Treelet restructuring where surface areas overflow float32 (every split of
a subset then costs the same: the first is kept), and at the primitive counts
where the builder changes its first tree (one workgroup up to 1,024)."""
import numpy as np
import pytest

import scenegen as sg
from oracle import build_ref as br


def _mesh(kind, n):
    m = sg.random_soup(n, 300 + n)
    # a power of two: the Morton keys do not change with it.  2^64: boxes of
    # triangles keep finite areas, those near the root overflow; 2^80: all do
    scale = {"finite": 0, "mixed": 64, "infinite": 80}[kind]
    m.verts = np.ldexp(np.asarray(m.verts, np.float32), scale)
    return m


def _definition(mesh, rounds):
    with np.errstate(over="ignore"):
        keys, ids = br.sort_pairs(br.morton_keys(mesh.verts, mesh.idx))
        lo, hi = br.tri_boxes(mesh.verts, mesh.idx)
        lo, hi = lo[ids], hi[ids]
        left, right, first, last = br.radix_tree(keys)
        blo, bhi = br.refit(lo, hi, first, last)
        return (lo, hi) + tuple(br.treelet_optimise(left, right, lo, hi, blo, bhi, rounds=rounds))


@pytest.mark.parametrize("kind", ["finite", "mixed", "infinite"])
@pytest.mark.parametrize("n", [3, 7, 8, 40])
def test_definition_is_a_tree(kind, n):
    lo, hi, L, R, BLO, BHI = _definition(_mesh(kind, n), 2)
    with np.errstate(over="ignore"):
        infinite = np.isinf(br.surface_area32(BLO, BHI))
    assert infinite.all() if kind == "infinite" else infinite[0] == (kind == "mixed")
    seen_leaf, seen_node, stack = np.zeros(n, int), np.zeros(n - 1, int), [0]
    while stack:
        x = stack.pop()
        seen_node[x] += 1
        box = []
        for c in (int(L[x]), int(R[x])):
            if c < 0:
                seen_leaf[-c - 1] += 1
                box.append((lo[-c - 1], hi[-c - 1]))
            else:
                stack.append(c)
                box.append((BLO[c], BHI[c]))
        assert np.array_equal(BLO[x], np.minimum(box[0][0], box[1][0]))
        assert np.array_equal(BHI[x], np.maximum(box[0][1], box[1][1]))
    assert (seen_leaf == 1).all() and (seen_node == 1).all()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["finite", "mixed", "infinite"])
@pytest.mark.parametrize("n", [2, 3, 7, 8, 40, 1023, 1024, 1025])
def test_restructuring_matches_definition(kind, n):
    import torch
    import paper_2001_09792_amd as rg
    from tests import bvh_check
    mesh = _mesh(kind, n)
    v = torch.from_numpy(np.ascontiguousarray(mesh.verts, np.float32)).cuda()
    i = torch.from_numpy(np.ascontiguousarray(mesh.idx, np.uint32).view(np.int32)).cuda()
    print(f"[treelet edges] {kind} {n}", flush=True)
    st = rg.lbvh_stages(v, i, builder="treelet", radius=2)
    _, _, L, R, BLO, BHI = _definition(mesh, 2)
    rank = br.leaf_order(L, R, n)
    relabel = lambda c: np.where(c < 0, -(rank[np.maximum(-c - 1, 0)] + 1), c).astype(np.int32)  # noqa: E731
    assert np.array_equal(st["left"].cpu().numpy(), relabel(L))
    assert np.array_equal(st["right"].cpu().numpy(), relabel(R))
    boxes = st["boxes"].cpu().numpy()
    assert np.array_equal(boxes[: n - 1, :3], BLO) and np.array_equal(boxes[: n - 1, 3:], BHI)
    for width in (2, 4, 8):
        b = rg.build_blas(v, i, None, width, 1, builder="treelet")
        bvh_check.check_blas(b.buf.cpu().numpy(), b.desc)
