"""Backward calls by the source of their anchors: a table from the prepare
launch (with the source gradient, or above 1024 tiles) or the tiles themselves,
and targets with SIP, whose tiles take their box from the positions.  Against
the FP64 oracle."""
import numpy as np
import pytest
import torch

from synth import configs, draw_sip
from tests.test_gpu_grad import INTERPS, _compare_wcs_grad

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dfr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_03932_amd as d
    return d


@pytest.mark.parametrize("interp", [1, 2])
@pytest.mark.parametrize("shape", [(1024, 1024), (1025, 1024)])  # 1024 and 1056 tiles of 32x32
def test_wcs_gradient_alone_on_both_sides_of_the_table(dfr, orc, interp, shape):
    c = configs.grad(size=1000)
    print(f"backward without source gradient interp={interp} shape={shape}", flush=True)
    src = torch.from_numpy(c.src).cuda()
    g = np.random.default_rng(3).normal(0, 1, shape).astype(np.float32)
    args = (src, c.src_wcs, c.tgt_wcs, shape, INTERPS[interp], torch.from_numpy(g).cuda())
    none, gw = dfr.reproject_backward(*args, want_src=False, tile=1)
    gs, gw_src = dfr.reproject_backward(*args, tile=1)
    _, gw_default = dfr.reproject_backward(*args, want_src=False)
    gs_only, no_wcs = dfr.reproject_backward(*args, want_wcs=False, tile=1)
    assert none is None and no_wcs is None and torch.equal(gs_only, gs)
    _, ref, _, ref_abs = orc.grad(c.src, c.src_wcs, c.tgt_wcs, shape, interp, g.astype(np.float64),
                                  want_src=False, want_abs=True)
    for w in (gw, gw_src, gw_default):
        _compare_wcs_grad(w.cpu().numpy(), ref, ref_abs)


# A target with SIP takes the chain from anchors, whose positions are within
# 2e-5 px of the exact ones where test_gpu_grad assumes 2e-6: a weight moves by
# up to 4e-5 and a source entry by 16 of them (6.4e-4 max|g|); an interpolant's
# derivative by about 1e-5 relative, with the FP32 sums 1.2e-5 of the terms' magnitudes.
TSIP_SRC_TOL = 1e-3
TSIP_WCS_TOL = 6e-5


@pytest.mark.parametrize("interp", [0, 1, 2])
@pytest.mark.parametrize("order,factor", [(2, 1.0), (3, 50.0), (9, 20.0)])
@pytest.mark.parametrize("want_src", [True, False])
def test_target_with_sip(dfr, orc, interp, order, factor, want_src):
    c = configs.grad(size=160)
    shape = (171, 165)
    a, b = draw_sip(order, 80.0, np.random.default_rng(17))
    tw = c.tgt_wcs.copy(a=a * factor, b=b * factor)
    print(f"backward target sip order={order} interp={interp} want_src={want_src}", flush=True)
    src = torch.from_numpy(c.src).cuda()
    g = np.random.default_rng(3).normal(0, 1, shape).astype(np.float32)
    for tile in (0, 1, 5):
        gs, gw = dfr.reproject_backward(src, c.src_wcs, tw, shape, INTERPS[interp],
                                        torch.from_numpy(g).cuda(), want_src=want_src, tile=tile)
        ogs, ref, _, ref_abs = orc.grad(c.src, c.src_wcs, tw, shape, interp, g.astype(np.float64),
                                        want_abs=True)
        assert (gs is not None) == want_src
        if want_src:
            tol = 1e-5 if interp == 0 else TSIP_SRC_TOL
            assert np.abs(gs.cpu().numpy() - ogs).max() <= tol * np.abs(g).max()
        if interp:
            _compare_wcs_grad(gw.cpu().numpy(), ref, ref_abs, tol=TSIP_WCS_TOL)
        else:
            assert not gw.any()
