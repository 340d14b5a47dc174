"""Short launches give each ray a group of lanes, long ones a lane per ray:
the same rays traced in one long call and in short calls have the same hits,
bit for bit (both visit the same units and settle ties by index)."""
import numpy as np
import pytest

import scenegen as sg
from tests.helpers import scene_from_meshes

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

N = 180000    # above two rays per resident group (131,072 at width 4, 65,536 at width 8)
CHUNKS = [1, 3, 63, 64, 65, 4097, 20000, 60000]


def _scene():
    """Instances of a soup, a torus and an icosphere, one mirrored, some with
    flags: masks of two kinds, flipped facing, culling disabled."""
    rng = np.random.default_rng(17)
    meshes = [sg.random_soup(3000, 5, 1.0, 0.1), sg.torus(40, 40, 1.0, 0.3), sg.icosphere(3)]
    xf = sg.random_instances(rng, 40, extent=6.0).reshape(-1, 3, 4)
    xf[3, :, 0] *= -1.0
    flags = np.where(np.arange(40) % 3 == 0, 0x01, 0x03).astype(np.uint32)
    flags[5] |= 1 << 9
    flags[6] |= 1 << 8
    sc = scene_from_meshes(meshes, xforms=xf, blas_id=(np.arange(40) % 3).astype(np.uint32),
                           inst_mat=np.zeros(40, np.uint32))
    return sc, flags


@pytest.mark.parametrize("width,leaf", [(4, 1), (4, 4), (4, 8), (8, 1), (8, 8)])
@pytest.mark.parametrize("options", [False, True])
def test_short_calls_equal_a_long_one(width, leaf, options):
    import paper_2001_09792_amd as rg
    sc, flags = _scene()
    tl = rg.upload_scene(sc, width, leaf, inst_flags=flags if options else None)
    opts = dict(cull=rg.RAY_CULL_BACK, mask=0x02) if options else {}
    rays = rg.rays_to_device(sg.random_rays(N, 23, extent=7.0))
    full = {k: v.clone() for k, v in rg.trace_closest(tl, rays, **opts).items()}
    f_found = {k: v for k, v in rg.alloc_hits(N).items() if k in ("inst", "prim")}
    f_occ = rg.trace_any(tl, rays, found=f_found, **opts).clone()
    assert 0.05 < float(f_occ.float().mean()) < 0.95
    at = 0
    for m in CHUNKS:
        r = rays[:, at:at + m].contiguous()
        h = rg.trace_closest(tl, r, **opts)
        for k in ("inst", "prim", "t", "u", "v"):
            assert bool((h[k] == full[k][at:at + m]).all()), (k, m)
        found = {k: v for k, v in rg.alloc_hits(m).items() if k in ("inst", "prim")}
        occ = rg.trace_any(tl, r, found=found, **opts)
        assert bool((occ == f_occ[at:at + m]).all()), m
        for k in found:
            assert bool((found[k] == f_found[k][at:at + m]).all()), (k, m)
        at += m
