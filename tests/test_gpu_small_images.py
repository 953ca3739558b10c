"""Tile shapes of small images: an image of a few tiles takes the shape whose
rounds of tiles take least.  Every shape the choice can take (width 64, 48, 32
or 16, heights 16 to 128, boxes sorted in LDS or in global scratch) is held
against the oracle, through the default route and at the shape itself, on
images that end inside a tile."""

import numpy as np
import pytest

import workloads
from oracle import footprints as OF

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mf():
    import paper_2505_22938_amd as m
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    m.lib()
    return m


def image(dtype, w, h, seed):
    return workloads.special_floats(w, h, seed) if dtype == "f32" else \
        workloads.uniform(w, h, dtype, seed)


@pytest.mark.parametrize("w,h,r", [(70, 45, 26), (130, 131, 24), (201, 90, 40), (90, 260, 64)])
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_default_route(mf, oracle_mod, dtype, w, h, r):
    img = image(dtype, w, h, r)
    got = mf.median_filter(torch.from_numpy(img).cuda(), mf.Footprint.disc(r), "mirror").cpu().numpy()
    exp = oracle_mod.filter(img, OF.disc(r), "mirror")
    assert np.array_equal(got.view(np.uint8), exp.view(np.uint8))


@pytest.mark.parametrize("tile", [(64, 128), (64, 48), (64, 16), (48, 32), (48, 80), (32, 48), (32, 16),
                                  (16, 16), (16, 80), (64, 64)])
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_shapes(mf, oracle_mod, dtype, tile):
    img = image(dtype, 150, 101, 5)
    dev = torch.from_numpy(img).cuda()
    for fp, ofp in ((mf.Footprint.disc(13), OF.disc(13)),
                    (mf.Footprint.ellipse(63, 20, 20), OF.ellipse(63, 20, 20))):
        mf.set_tile_override(*tile)
        try:
            got = mf.median_filter(dev, fp, "clamp").cpu().numpy()
        finally:
            mf.set_tile_override(0, 0)
        exp = oracle_mod.filter(img, ofp, "clamp")
        assert np.array_equal(got.view(np.uint8), exp.view(np.uint8)), fp
