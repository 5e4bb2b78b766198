"""Cells of a batch frame that a bound tells apart as out of reach get no
model.  Frames all over (and far off) the target grid, rotated, scaled, with
source SIP of every order, steep SIP and from behind the sky: every frame of
the batch, dense and cropped, must equal the single-image call, which models
every cell, bit for bit; and its box must contain every covered pixel."""
import numpy as np
import pytest
import torch

from synth import WcsParams, configs, draw_sip, fit_inverse_sip

pytestmark = pytest.mark.gpu
SHAPE = (700, 1100)


@pytest.fixture(scope="module")
def dfr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_03932_amd as d
    return d


def _frames(order, factor):
    """One frame per geometry: (image, WCS)."""
    rng = np.random.default_rng(100 * order + 7)
    s = 2.85 / 3600.0
    frames = []
    for k, (dx, dy) in enumerate([(0, 0), (-500, 300), (540, -350), (700, 0), (0, 520), (900, 900),
                                  (-2000, 40), (20000, 0)]):
        h, w = int(rng.integers(40, 300)), int(rng.integers(40, 300))
        rot, scale = rng.uniform(-180, 180), rng.uniform(0.5, 2.0)
        crval = ((150.0 + dx * s) % 360.0, 2.0 + dy * s)
        src = (100 + rng.standard_normal((h, w))).astype(np.float32)
        sw = WcsParams.tan(crval, 2.85 * scale, rot, (h, w))
        if order:
            a, b = draw_sip(min(order, 6), 0.5 * max(h, w), rng)
            a, b = factor * a, factor * b
            ap, bp, _ = fit_inverse_sip(a, b, order, sw.crpix, (h, w))
            sw = sw.copy(a=a, b=b, ap=ap, bp=bp)
        frames.append((src, sw))
    src, sw = frames[0]
    frames.append((src, sw.copy(crval=(330.0, -2.0))))  # the far side of the sky
    return frames


@pytest.mark.parametrize("interp", ["nearest", "bilinear", "bicubic"])
@pytest.mark.parametrize("order,factor", [(0, 1.0), (2, 1.0), (3, 300.0), (5, 30.0), (6, 1.0), (9, 300.0)])
def test_frames_equal_single_calls(dfr, order, factor, interp):
    print(f"reach order={order} factor={factor} interp={interp}", flush=True)
    _compare(dfr, order, factor, interp, SHAPE)


@pytest.mark.parametrize("shape", [(2200, 3000), (300, 40000), (2049, 257)])
def test_blocks_of_larger_grids(dfr, shape):
    print(f"reach shape={shape}", flush=True)
    _compare(dfr, 3, 30.0, "bilinear", shape)


def _compare(dfr, order, factor, interp, SHAPE):
    frames = _frames(order, factor)
    tw = configs.plain().tgt_wcs.copy(crpix=(SHAPE[1] / 2, SHAPE[0] / 2))
    srcs = [torch.from_numpy(s).cuda() for s, _ in frames]
    wcss = [w for _, w in frames]
    outs, fps = dfr.reproject_batch(srcs, wcss, tw, SHAPE, interp)
    co, cf, boxes = dfr.reproject_batch_cropped(srcs, wcss, tw, SHAPE, interp)
    for i, (src, w) in enumerate(zip(srcs, wcss)):
        o, f = dfr.reproject(src, w, tw, SHAPE, interp)
        assert torch.equal(outs[i], o) and torch.equal(fps[i], f), i
        x0, y0, bw, bh = boxes[i]
        inside = torch.zeros(SHAPE, dtype=torch.bool, device="cuda")
        inside[y0:y0 + bh, x0:x0 + bw] = True
        assert not (f > 0)[~inside].any(), i
        assert torch.equal(co[i], o[y0:y0 + bh, x0:x0 + bw]), i
        assert torch.equal(cf[i], f[y0:y0 + bh, x0:x0 + bw]), i
