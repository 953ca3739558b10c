"""Sorts of boxes too large for LDS tiles: chunks of 16 bytes that end in the
box or across the image's edge, images narrower than a chunk, rows at any
address, equal keys by the thousand, float words that just fit LDS and that do
not (override), all against the oracle."""

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


def image(dtype, kind, w, h, seed):
    if kind == "flat":
        img = workloads.uniform(w, h, "u8", seed) // 128
        return img.astype({"u8": np.uint8, "u16": np.uint16, "f32": np.float32}[dtype])
    return workloads.special_floats(w, h, seed) if dtype == "f32" else \
        workloads.uniform(w, h, dtype, seed)


@pytest.mark.parametrize("kind", ["uniform", "flat"])
# (tile, window radii: box 160 x 224 in LDS for float32, 201 x 217 not)
@pytest.mark.parametrize("tile,rx,ry", [((64, 128), 48, 48), ((61, 117), 70, 50), ((54, 56), 100, 100),
                                        ((7, 90), 100, 61)])
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_against_oracle(mf, oracle_mod, dtype, tile, rx, ry, kind):
    fp, ofp = (mf.Footprint.disc(rx), OF.disc(rx)) if rx == ry else \
        (mf.Footprint.ellipse(rx, ry, 0), OF.ellipse(rx, ry, 0))
    for w, h, pad in ((131, 137, 3), (3, 40, 0), (18, 9, 1)):
        img = image(dtype, kind, w, h, rx)
        wide = torch.zeros((h, w + pad), dtype=torch.from_numpy(img).dtype, device="cuda")
        wide[:, pad:].copy_(torch.from_numpy(img).cuda())
        mf.set_tile_override(*tile)
        try:
            got = mf.median_filter(wide[:, pad:], fp, "mirror").contiguous().cpu().numpy()
        finally:
            mf.set_tile_override(0, 0)
        exp = oracle_mod.filter(img, ofp, "mirror")
        assert np.array_equal(got.view(np.uint8), exp.view(np.uint8)), (w, h)
