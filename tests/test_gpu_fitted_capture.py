"""A call whose fitted shape needs scratch that a capturing stream cannot get
runs on the default shape instead: captured without an earlier call on the
stream, replayed, and equal to the eager call."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mf():
    import paper_2505_22938_amd as m
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    m.lib()
    return m


@pytest.mark.parametrize("call", ["plain", "ranks", "windows"])
@pytest.mark.parametrize("dtype,w,h,r", [("u16", 2048, 2048, 48), ("f32", 2048, 2048, 40)])
def test_captured_on_a_fresh_stream(mf, dtype, w, h, r, call):
    img = torch.from_numpy(workloads.special_floats(w, h, 1) if dtype == "f32" else
                           workloads.uniform(w, h, dtype, 1)).cuda()
    fps = [mf.Footprint.disc(r), mf.Footprint.disc(r - 1)]
    outs = [torch.empty_like(img) for _ in range(2)]

    def run():
        if call == "plain":
            mf.median_filter(img, fps[0], "clamp", out=outs[0])
        elif call == "ranks":
            mf.rank_filter(img, fps[0], [5, fps[0].taps // 2], "clamp", outs=outs)
        else:
            mf.window_filter(img, fps, "clamp", outs=outs)

    run()          # span tables and the current stream's scratch
    torch.cuda.synchronize()
    n = 1 if call == "plain" else 2
    exp = [o.cpu().numpy().view(np.uint8) for o in outs[:n]]
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        run()
    for _ in range(3):
        for o in outs:
            o.copy_(torch.zeros_like(o))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for o, e in zip(outs[:n], exp):
            assert np.array_equal(o.cpu().numpy().view(np.uint8), e)
