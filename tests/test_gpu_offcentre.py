"""Tile engine under windows that do not contain their centre pixel: a window
wholly to one side of it puts the window centres of a tile's first columns
or rows outside the tile's input box."""

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


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("verts", [[(3, 3), (9, 3), (9, 8), (3, 8)],
                                   [(3, -3), (9, -3), (9, 3), (3, 3)],
                                   [(-3, 3), (3, 3), (3, 9), (-3, 9)],
                                   [(-9, -8), (-3, -8), (-3, -3), (-9, -3)]])
def test_windows_beside_their_centre(mf, oracle_mod, dtype, verts):
    img = workloads.uniform(90, 70, dtype, 3)
    exp = oracle_mod.filter(img, OF.polygon(verts), "mirror")
    mf.set_tile_override(32, 32)
    try:
        got = mf.median_filter(torch.from_numpy(img).cuda(), mf.Footprint.polygon(verts), "mirror")
        torch.cuda.synchronize()
    finally:
        mf.set_tile_override(0, 0)
    assert np.array_equal(got.cpu().numpy().view(np.uint8), exp.view(np.uint8))
