"""Captured calls and the scratch of their stream.  Windows whose default tiles
sort in LDS take no scratch into a graph, so graphs captured on one warmed
stream replay on several streams at once, beside eager calls on it and after
mf_release_scratch; and a stream warmed by a call on a larger image can be
captured on a smaller one whatever shapes the two fit.  Two host threads on one
stream may each need its scratch grown."""

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


def image(dtype, w, h, seed):
    return torch.from_numpy(workloads.special_floats(w, h, seed) if dtype == "f32" else
                            workloads.uniform(w, h, dtype, seed)).cuda()


def same(a, b):
    return np.array_equal(a.cpu().numpy().view(np.uint8), b.cpu().numpy().view(np.uint8))


def call(mf, kind, img, fps, outs):
    if kind == "plain":
        mf.median_filter(img, fps[0], "clamp", out=outs[0])
    elif kind == "ranks":
        mf.rank_filter(img, fps[0], [5, fps[0].taps // 2], "clamp", outs=outs)
    else:
        mf.window_filter(img, fps, "clamp", outs=outs)


@pytest.mark.parametrize("kind", ["plain", "ranks", "windows"])
@pytest.mark.parametrize("dtype,r", [("u8", 46), ("u16", 48), ("f32", 40)])
def test_graphs_of_one_stream_at_once(mf, dtype, r, kind):
    n = 1 if kind == "plain" else 2
    big = image("f32", 2048, 2048, 4)
    big_out, big_fp = torch.empty_like(big), mf.Footprint.disc(90)
    mf.median_filter(big, big_fp, "clamp", out=big_out)   # its table
    mf.release_scratch()   # (torch hands out its streams again and again)
    fps = [mf.Footprint.disc(r), mf.Footprint.disc(r - 1)]
    imgs = [image(dtype, 2048, 2048, s) for s in (1, 2, 3)]
    outs = [[torch.empty_like(imgs[0]) for _ in range(n)] for _ in imgs]
    home, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(home):            # tables, and whatever scratch eager calls take
        for im, o in zip(imgs, outs):
            call(mf, kind, im, fps, o)
    torch.cuda.synchronize()
    exp = [[p.clone() for p in o] for o in outs]
    graphs = []
    for im, o in zip(imgs[:2], outs):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=home):
            call(mf, kind, im, fps, o)
        graphs.append(g)

    def check(k):
        torch.cuda.synchronize()
        for o, e in zip(outs[:k], exp):
            for a, b in zip(o, e):
                assert same(a, b)
                a.copy_(torch.zeros_like(a))
        torch.cuda.synchronize()

    # the graphs hold nothing of the stream's scratch: a larger buffer replaces
    # it (one that a graph may use is kept beside), and it can be released
    def released_after_big(stream):
        with torch.cuda.stream(stream):
            mf.median_filter(big, big_fp, "clamp", out=big_out)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        mf.release_scratch()
        return torch.cuda.mem_get_info()[0] - free

    with_graphs = released_after_big(home)
    assert with_graphs <= released_after_big(other) + (4 << 20)
    check(3)
    for _ in range(3):
        with torch.cuda.stream(other):
            graphs[0].replay()
        with torch.cuda.stream(home):
            graphs[1].replay()
        check(2)
    for _ in range(3):
        with torch.cuda.stream(other):
            graphs[0].replay()
        with torch.cuda.stream(home):
            call(mf, kind, imgs[2], fps, outs[2])
        torch.cuda.synchronize()
        assert all(same(a, b) for a, b in zip(outs[0], exp[0]))
        assert all(same(a, b) for a, b in zip(outs[2], exp[2]))


@pytest.mark.parametrize("dtype,r,a,b", [("u16", 100, (641, 479), (400, 300)),
                                         ("u16", 64, (1200, 1100), (1024, 1024)),
                                         ("u16", 64, (1500, 1200), (641, 479)),
                                         ("f32", 64, (1200, 900), (800, 800)),
                                         ("f32", 100, (641, 479), (400, 300)),
                                         ("f32", 48, (3840, 2160), (500, 301)),
                                         ("u8", 68, (558, 624), (458, 609))])
def test_captured_after_a_larger_image(mf, dtype, r, a, b):
    mf.release_scratch()
    fp = mf.Footprint.disc(r)
    large, small = image(dtype, *a, 1), image(dtype, *b, 2)
    out = torch.empty_like(small)
    exp = mf.median_filter(small, fp, "mirror")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        mf.median_filter(large, fp, "mirror")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        mf.median_filter(small, fp, "mirror", out=out)
    for _ in range(3):
        out.copy_(torch.zeros_like(out))
        g.replay()
        torch.cuda.synchronize()
        assert same(out, exp)
    del g
    torch.cuda.synchronize()
    mf.release_scratch()


@pytest.mark.parametrize("dtype,r", [("u16", 48), ("f32", 40)])
def test_per_thread_stream(mf, dtype, r):
    """One handle names a stream of each host thread, so middle windows keep their
    LDS tiles there too."""
    import ctypes
    img, fp = image(dtype, 2048, 2048, 1), mf.Footprint.disc(r)
    code = {"u16": 1, "f32": 2}[dtype]
    assert mf.query_call(2048, 2048, code, fp)["scratch_bytes"] > 0
    exp = mf.median_filter(img, fp, "clamp")
    out = torch.empty_like(img)
    torch.cuda.synchronize()
    mf.release_scratch()
    P = ctypes.c_void_p
    rc = mf.lib().median_filter(P(img.data_ptr()), 2048, 2048, 2048 * img.element_size(), code,
                                fp.handle, 0, P(out.data_ptr()), P(2))   # hipStreamPerThread
    assert rc == 0
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    mf.release_scratch()
    assert torch.cuda.mem_get_info()[0] - free < (1 << 20)
    assert same(out, exp)


def test_captured_without_an_earlier_call_is_refused(mf):
    """Global-scratch windows on a stream that no call has used, or whose scratch
    was released."""
    img, fp = image("u16", 2048, 2048, 1), mf.Footprint.disc(64)
    mf.median_filter(img, fp, "clamp")   # the table
    out = torch.empty_like(img)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        mf.median_filter(img, fp, "clamp")
    torch.cuda.synchronize()
    mf.release_scratch()
    status = None
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        out.copy_(img)
        try:
            mf.median_filter(img, fp, "clamp", out=out)
        except mf.MedianFilterError as e:
            status = e.status
    assert status == -3


def test_two_threads_on_one_stream(mf):
    """One thread's calls use the stream's scratch while the other's make it grow
    again and again."""
    import threading
    small, sfp = image("u16", 2048, 2048, 1), mf.Footprint.disc(46)
    big = image("f32", 900, 700, 2)
    radii = (52, 58, 64, 70, 76, 82, 90, 100)
    bfps = [mf.Footprint.disc(r) for r in radii]
    exp = mf.median_filter(small, sfp, "clamp")
    bexp = [mf.median_filter(big, fp, "clamp") for fp in bfps]
    assert mf.query_call(2048, 2048, mf.MF_U16, sfp)["path"] == "scratch"
    s = torch.cuda.Stream()
    outs = [torch.empty_like(small) for _ in range(40)]
    bouts = [torch.empty_like(big) for _ in radii]
    torch.cuda.synchronize()
    mf.release_scratch()
    errors = []

    def run(calls):
        try:
            for call in calls:
                call()
        except Exception as e:   # noqa: BLE001
            errors.append(e)

    a = threading.Thread(target=run, args=([lambda o=o: mf.median_filter(small, sfp, "clamp", out=o,
                                                                         stream=s) for o in outs],))
    b = threading.Thread(target=run, args=([lambda f=f, o=o: mf.median_filter(big, f, "clamp", out=o,
                                                                              stream=s)
                                            for f, o in zip(bfps, bouts)],))
    a.start()
    b.start()
    a.join()
    b.join()
    torch.cuda.synchronize()
    assert not errors, errors
    assert all(same(o, exp) for o in outs)
    assert all(same(o, e) for o, e in zip(bouts, bexp))
    mf.release_scratch()
