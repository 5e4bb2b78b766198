"""Calls on a stream under capture, on the device: what is refused is refused
without harm to the capture or to later calls, and what is recorded keeps no
pointer into scratch that a later call may move."""
import pytest
import torch

from synth import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dfr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_03932_amd as d
    return d


@pytest.mark.parametrize("kind", ["batch", "coadd", "cropped"])
def test_stack_calls_are_refused(dfr, kind):
    c = configs.sip3(scale=0.06)
    src = torch.from_numpy(c.src).cuda()
    shape = c.out_shape
    boxes = [[0, 0, shape[1], shape[0]]]
    outs, a, b = [torch.zeros(shape, device="cuda")], *torch.zeros((2, *shape), device="cuda")

    def run():
        if kind == "coadd":
            dfr.coadd_batch([src], [c.src_wcs], c.tgt_wcs, shape, sum_wf=a, sum_f=b, coadd=False)
            return a
        if kind == "batch":
            return dfr.reproject_batch([src], [c.src_wcs], c.tgt_wcs, shape, outs=outs,
                                       footprint=False)[0][0]
        return dfr.reproject_batch_cropped([src], [c.src_wcs], c.tgt_wcs, shape, boxes=boxes,
                                           footprint=False)[0][0]

    print(f"capture of a stack call kind={kind}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for _ in range(5):
            want = run().clone()
    torch.cuda.synchronize()
    mark = torch.zeros(8, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        mark.add_(1.0)
        with pytest.raises(dfr.DfrError):
            run()
    for _ in range(3):
        g.replay()
    torch.cuda.synchronize()
    assert torch.equal(mark, torch.full_like(mark, 3.0))
    with torch.cuda.stream(stream):
        for _ in range(5):
            assert torch.equal(run(), want)
    assert want.abs().max() > 0


def test_target_with_sip_after_a_warm_up(dfr):
    """The warm-up leaves a workspace that would hold the models' table; a
    larger call after the capture frees it.  The graph uses neither."""
    from synth import draw_sip
    import numpy as np
    c = configs.sip3(scale=0.06)
    a, b = draw_sip(3, 180.0, np.random.default_rng(21))
    tw = c.tgt_wcs.copy(a=a * 50.0, b=b * 50.0)
    src = torch.from_numpy(c.src).cuda()
    call = lambda **k: dfr.reproject(src, c.src_wcs, tw, c.out_shape, "bilinear", **k)
    want, want_fp = call(precision="f32_anchor")
    out, fp = torch.zeros_like(want), torch.zeros_like(want)
    print("capture of a target with SIP on a used stream", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call(out=out, fp=fp)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        call(out=out, fp=fp)
    with torch.cuda.stream(stream):  # a much larger table and integer image
        dfr.reproject_backward(src, c.src_wcs, c.tgt_wcs, (3000, 3000), "bilinear",
                               torch.ones((3000, 3000), device="cuda"))
    torch.cuda.synchronize()
    for _ in range(3):
        out.zero_()
        fp.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(fp, want_fp)
