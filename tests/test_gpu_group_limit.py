"""Numbers of rays on both sides of the most that get a group of lanes each:
two rays per resident group at width 4, two and a quarter at width 8, with the
default launch parameters and with more waves asked for than stay resident.
The same rays have the same hits, and a frame the same image, on either path."""
import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _limits(width):
    groups = torch.cuda.get_device_properties(0).multi_processor_count * 16 * (64 // width)
    return [2 * groups, 2 * groups + groups // 4, 2 * groups + groups // 2]


@pytest.mark.parametrize("waves", [16, 64])
@pytest.mark.parametrize("width", [4, 8])
def test_hits_around_the_limit(width, waves):
    import paper_2001_09792_amd as rg
    tl = rg.upload_scene(sg.config_two_level(seed=1), width, 1)
    most = max(_limits(width)) + 1
    rays = rg.rays_to_device(sg.random_rays(most, 29, extent=20.0))
    want = {k: [] for k in ("inst", "prim", "t")}
    occ_want = []
    for at in range(0, most, 20011):  # short calls: groups
        r = rays[:, at:at + 20011].contiguous()
        h = rg.trace_closest(tl, r)
        for k in want:
            want[k].append(h[k].clone())
        occ_want.append(rg.trace_any(tl, r).clone())
    want = {k: torch.cat(v) for k, v in want.items()}
    occ_want = torch.cat(occ_want)
    saved = rg.trace_tuning(scope="trace")
    try:
        rg.trace_tuning(waves_per_cu=waves, scope="trace")
        for n in (m + d for m in _limits(width) for d in (-1, 0, 1)):
            print(f"[group limit] W={width} waves {waves} n={n}", flush=True)
            r = rays[:, :n].contiguous()
            h = rg.trace_closest(tl, r)
            for k in want:
                assert bool((h[k] == want[k][:n]).all()), (k, n)
            assert bool((rg.trace_any(tl, r) == occ_want[:n]).all()), n
    finally:
        rg.trace_tuning(scope="trace", **saved)


@pytest.mark.parametrize("width", [4, 8])
def test_frames_around_the_limit(width):
    import paper_2001_09792_amd as rg
    sc = sg.config_two_level(seed=1, max_depth=1)
    tl = rg.upload_scene(sc, width, 1)
    saved = rg.trace_tuning(scope="frame")
    for m in _limits(width):
        h = 256
        for w in (m // h, m // h + 1):
            print(f"[group limit] W={width} frame {w}x{h}", flush=True)
            img = rg.render(tl, sc.materials, sc.camera, sc.light, w, h, 1).clone()
            try:
                rg.trace_tuning(waves_per_cu=4, scope="frame")  # fewer groups: a lane per ray
                lanes = rg.render(tl, sc.materials, sc.camera, sc.light, w, h, 1).clone()
            finally:
                rg.trace_tuning(scope="frame", **saved)
            assert torch.equal(img, lanes)
            assert float(img.std()) > 0.01
    assert np.isfinite(img.cpu().numpy()).all()
