"""Windows too wide for a tile's box are refused by every call, also flat ones
of few enough taps for the bit planes; the widest window a box holds is not."""

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


def rect(w, h):
    x, y = -(w // 2), -(h // 2)
    return [(x, y), (x + w - 1, y), (x + w - 1, y + h - 1), (x, y + h - 1)]


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("w,h", [(249, 2), (300, 2), (300, 5), (500, 3)])
def test_refused(mf, dtype, w, h):
    img = torch.from_numpy(workloads.uniform(70, 40, dtype, 1)).cuda()
    out = torch.empty_like(img)
    fp = mf.Footprint.polygon(rect(w, h))
    for call in (lambda: mf.median_filter(img, fp, out=out),
                 lambda: mf.median_filter(img, fp, out=out, rank=3),
                 lambda: mf.median_filter_noalloc(img, fp, out),
                 lambda: mf.rank_filter(img, fp, [1, 2]),
                 lambda: mf.window_filter(img, [fp, mf.Footprint.disc(2)]),
                 lambda: mf.BatchPlan([(img, out, fp, "clamp")])):
        with pytest.raises(mf.MedianFilterError) as e:
            call()
        assert e.value.status == -3


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_widest(mf, oracle_mod, dtype):
    img = workloads.uniform(70, 40, dtype, 1)
    for h in (2, 6):
        v = rect(248, h)
        got = mf.median_filter(torch.from_numpy(img).cuda(), mf.Footprint.polygon(v), "mirror")
        exp = oracle_mod.filter(img, OF.polygon(v), "mirror")
        assert np.array_equal(got.cpu().numpy().view(np.uint8), exp.view(np.uint8)), h
