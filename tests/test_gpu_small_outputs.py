"""Outputs of few tiles take one launch whose groups make the models of their
own cells; above the line, and in a plan, a table holds them.  Same bits on
both sides of the line, for every source order the one-launch form covers and
the first it does not."""
import numpy as np
import pytest
import torch

from synth import WcsParams, configs, draw_sip, fit_inverse_sip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dfr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_03932_amd as d
    return d


def _case(order):
    c = configs.plain(size=300)
    if not order:
        return c.src, c.src_wcs, c.tgt_wcs
    a, b = draw_sip(min(order, 4), 150.0, np.random.default_rng(order))
    ap, bp, _ = fit_inverse_sip(50 * a, 50 * b, order, c.src_wcs.crpix, (300, 300))
    return c.src, c.src_wcs.copy(a=50 * a, b=50 * b, ap=ap, bp=bp), c.tgt_wcs


@pytest.mark.parametrize("interp", ["nearest", "bilinear", "bicubic"])
@pytest.mark.parametrize("order", [0, 1, 2, 3, 4, 5, 6])
def test_same_bits_as_a_plan(dfr, order, interp):
    s, sw, tw = _case(order)
    src = torch.from_numpy(s).cuda()
    # 1, 767, 768 and 769 tiles of 32x32; 64x16 tiles; a ragged shape
    for shape in [(1, 1), (767 * 32, 32), (32 * 32, 24 * 32), (769 * 32, 32), (300, 301), (33, 65)]:
        print(f"small order={order} interp={interp} shape={shape}", flush=True)
        o, f = dfr.reproject(src, sw, tw, shape, interp, nan_outside=True)
        with dfr.Plan(src.shape, sw, tw, shape, interp, nan_outside=True) as plan:
            po, pf = plan.execute(src)
        assert torch.equal(torch.nan_to_num(o, nan=-7.0), torch.nan_to_num(po, nan=-7.0))
        assert torch.equal(f, pf)
        for tile in (1, 4, 7, 10):
            o2, f2 = dfr.reproject(src, sw, tw, shape, interp, nan_outside=True, tile=tile)
            assert torch.equal(f2, f) and torch.equal(torch.isnan(o2), torch.isnan(o))
            assert torch.equal(torch.nan_to_num(o2), torch.nan_to_num(o)), tile
    # debug positions through the one-launch form: the same as through the anchors within 2e-5
    p = dfr.reproject(src, sw, tw, (300, 301), interp, debug_positions=True)[2]
    q = dfr.reproject(src, sw, tw, (300, 301), interp, precision="f32_anchor", debug_positions=True)[2]
    if interp != "nearest":
        assert (p - q).abs().nan_to_num().max().item() <= 2e-5


@pytest.mark.parametrize("interp", ["nearest", "bilinear", "bicubic"])
def test_order_5_around_its_own_limit(dfr, interp):
    s, sw, tw = _case(5)
    src = torch.from_numpy(s).cuda()
    for shape in [(511 * 32, 32), (16 * 32, 32 * 32), (513 * 32, 32)]:  # 511, 512 and 513 tiles
        print(f"small order 5 interp={interp} shape={shape}", flush=True)
        o, f = dfr.reproject(src, sw, tw, shape, interp)
        with dfr.Plan(src.shape, sw, tw, shape, interp) as plan:
            po, pf = plan.execute(src)
        assert torch.equal(o, po) and torch.equal(f, pf) and f.any()
