"""The backward's tiles whose box comes from the anchors' bounds: interior ones
take no per-pixel test, and every thread's run of output gradients is one load
at any alignment.  Compared bit for bit with the same call where only the
alignment, the tile shape or values under a zero gradient differ."""
import numpy as np
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


@pytest.mark.parametrize("interp", ["nearest", "bilinear", "bicubic"])
def test_values_under_a_zero_gradient(dfr, interp):
    """A zero output gradient masks whatever the pixel's taps hold."""
    c = configs.grad(size=200)
    src = torch.from_numpy(c.src).cuda()
    gen = torch.Generator(device="cuda").manual_seed(3)
    g = torch.randn(c.out_shape, device="cuda", generator=gen)
    bad = src.clone()
    bad[90:97, 80:99] = float("nan")
    bad[120, 60] = float("inf")
    out, _ = dfr.reproject(bad, c.src_wcs, c.tgt_wcs, c.out_shape, interp)
    touched = torch.nn.functional.max_pool2d((~torch.isfinite(out)).float()[None, None], 3, 1, 1)[0, 0] > 0
    assert 0 < touched.sum() < 2000
    g[touched] = 0.0
    print(f"zero gradient interp={interp}", flush=True)
    want = dfr.reproject_backward(src, c.src_wcs, c.tgt_wcs, c.out_shape, interp, g)
    got = dfr.reproject_backward(bad, c.src_wcs, c.tgt_wcs, c.out_shape, interp, g)
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


@pytest.mark.parametrize("interp", ["bilinear", "bicubic"])
@pytest.mark.parametrize("shape", [(1, 1), (5, 3), (33, 66), (70, 129), (64, 128)])
def test_gradient_at_any_alignment(dfr, interp, shape):
    c = configs.grad(size=160)
    src = torch.from_numpy(c.src).cuda()
    buf = torch.randn(shape[0] * shape[1] + 8, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(5))
    ref = None
    for offset in range(4):
        print(f"gradient interp={interp} shape={shape} offset={offset}", flush=True)
        view = buf[offset:offset + shape[0] * shape[1]].view(shape)
        view.copy_(buf[:shape[0] * shape[1]].view(shape).clone() if ref is None else ref[2])
        gs, gw = dfr.reproject_backward(src, c.src_wcs, c.tgt_wcs, shape, interp, view)
        if ref is None:
            ref = (gs, gw, view.clone())
        assert torch.equal(gs, ref[0]) and torch.equal(gw, ref[1])


@pytest.mark.parametrize("interp", ["nearest", "bilinear", "bicubic"])
def test_tile_shapes_mix_interior_and_edge_tiles(dfr, interp):
    """Source smaller than the target: interior, edge, half-covered and empty
    tiles; the source adjoint is exact, so every tile shape gives its bits."""
    c = configs.grad(size=150)
    src = torch.from_numpy(c.src).cuda()
    shape = (260, 300)
    tw = c.tgt_wcs.copy(crpix=(c.tgt_wcs.crpix[0] + 70, c.tgt_wcs.crpix[1] + 60))
    g = torch.randn(shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(9))
    ref = None
    for tile in (1, 2, 4, 5, 8, 10):
        print(f"tiles interp={interp} tile={tile}", flush=True)
        gs, gw = dfr.reproject_backward(src, c.src_wcs, tw, shape, interp, g, tile=tile)
        ref = (gs, gw) if ref is None else ref
        assert torch.equal(gs, ref[0])
        assert torch.allclose(gw, ref[1], rtol=1e-4, atol=1e-5 * float(ref[1].abs().max()))
    assert float(ref[0].abs().max()) > 0


def test_nearest_nan_gradient_on_any_tile(dfr):
    """The adjoint's integers do not depend on the tile shape, of a gradient
    that is not finite neither: interior and edge tiles form the same ones."""
    c = configs.grad(size=150)
    src = torch.from_numpy(c.src).cuda()
    shape = (260, 300)
    tw = c.tgt_wcs.copy(crpix=(c.tgt_wcs.crpix[0] + 70, c.tgt_wcs.crpix[1] + 60))
    g = torch.randn(shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(9))
    g[::9, ::7] = float("nan")
    ref = None
    for tile in (1, 2, 4, 5, 8, 10):
        print(f"nearest NaN gradient tile={tile}", flush=True)
        gs, _ = dfr.reproject_backward(src, c.src_wcs, tw, shape, "nearest", g, tile=tile)
        ref = gs if ref is None else ref
        assert torch.equal(gs, ref)
    clean = dfr.reproject_backward(src, c.src_wcs, tw, shape, "nearest", g.nan_to_num(0.0))[0]
    assert 0 < (ref != clean).sum() < ref.numel() // 20


@pytest.mark.parametrize("want_src", [True, False])
def test_masked_bicubic_gradient_is_passed_over(dfr, want_src):
    """Waves whose output gradient is all zero do no tap work: a call without
    any takes under three quarters of a full one (0.6 where they are passed
    over, 0.9 where they are not), and nothing comes of it."""
    c = configs.grad(size=2048)
    src = torch.from_numpy(c.src).cuda()
    g = torch.randn(c.out_shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))

    def best(grad):
        t = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                out = dfr.reproject_backward(src, c.src_wcs, c.tgt_wcs, c.out_shape, "bicubic", grad,
                                             want_src=want_src)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        return min(t), out

    print(f"masked gradient want_src={want_src}", flush=True)
    full, _ = best(g)
    none, (gs, gw) = best(torch.zeros_like(g))
    print("full, none (us)", 50 * full, 50 * none)
    assert none < 0.75 * full
    assert (gs is None or not gs.any()) and not gw.any()
