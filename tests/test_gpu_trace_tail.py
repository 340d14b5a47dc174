"""A trace call writes the results of its own rays and nothing past them,
whatever the number of rays in its last packet (the kernels gather results
per packet and write them out by a mask of finished rays)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]

import paper_2001_09792_amd as rg  # noqa: E402
import scenegen as sg  # noqa: E402

ROOM = 128  # entries of each output buffer past the call's rays


@pytest.fixture(scope="module")
def scene():
    return rg.upload_scene(sg.config_small())


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 40, 48, 56, 63, 64, 65, 100, 1000, 4129, 70000, 130001])
def test_results_end_with_the_rays(scene, n):
    rays = rg.rays_to_device(sg.random_rays(n, 11, extent=3.0))
    mark = {"t": 7.0, "u": 7.0, "v": 7.0, "inst": 7777, "prim": 7777}
    full = {k: torch.full_like(v, mark[k]) for k, v in rg.alloc_hits(n + ROOM).items()}
    got = rg.trace_closest(scene, rays, out={k: v[:n] for k, v in full.items()})
    occ = torch.full((n + ROOM,), 7, dtype=torch.uint8, device="cuda")
    found = {k: torch.full((n + ROOM,), 7777, dtype=torch.int32, device="cuda") for k in ("inst", "prim")}
    rg.trace_any(scene, rays, occluded=occ[:n], found={k: v[:n] for k, v in found.items()})
    for k, v in full.items():
        assert bool((v[n:] == mark[k]).all()), k
        assert not bool((v[:n] == mark[k]).any()), k
    assert bool((occ[n:] == 7).all()) and not bool((occ[:n] == 7).any())
    assert all(bool((v[n:] == 7777).all()) and not bool((v[:n] == 7777).any()) for v in found.values())
    hit = (got["inst"] != -1).cpu().numpy()
    np.testing.assert_array_equal(hit, occ[:n].cpu().numpy() != 0)
    # every ray alone in a call of its own gives the same hit
    for i in sorted({0, n // 2, n - 1}):
        one = rg.trace_closest(scene, rays[:, i:i + 1].contiguous())
        for k in ("t", "inst", "prim", "u", "v"):
            assert bool((one[k] == got[k][i:i + 1]).all()), (i, k)
