"""A frame starts each pixel's sums with its camera ray's own contribution,
also where that is none (a mirror, glass): what the scratch held before, an
earlier frame or arbitrary bytes, does not show."""
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth", [0, 1, 3])
@pytest.mark.parametrize("size", [(1, 1), (65, 33), (256, 144)])
def test_scratch_contents_do_not_show(depth, size):
    import paper_2001_09792_amd as rg
    W, H = size
    sc = sg.config_two_level(width=64, height=36)
    tl = rg.upload_scene(sc)
    r = rg.Renderer(W, H, depth)
    args = (tl, sc.materials, sc.camera, sc.light)
    r.scratch.zero_()
    want = r.render(*args).clone()
    again = r.render(*args).clone()      # over its own sums
    r.scratch.fill_(0xFF)
    dirty = r.render(*args).clone()
    assert float(want.sum()) > 0.0
    assert torch.equal(want, again) and torch.equal(want, dirty)
