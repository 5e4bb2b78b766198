"""The default tile follows the output's size and row alignment; results do
not: around each line of the rule every default equals an explicit tile."""
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


# one million and eight million pixels, rows of whole 128-byte lines or not
SHAPES = [(1024, 1024), (1024, 1056), (1023, 1025), (2048, 4096), (2049, 4096), (2047, 4099),
          (2050, 4099), (1, 70), (40, 32)]


@pytest.mark.parametrize("interp", ["nearest", "bilinear", "bicubic"])
@pytest.mark.parametrize("shape", SHAPES)
def test_default_equals_explicit(dfr, interp, shape):
    c = configs.sip3(scale=0.2)
    src = torch.from_numpy(c.src).cuda()
    print(f"default tile interp={interp} shape={shape}", flush=True)
    o, f = dfr.reproject(src, c.src_wcs, c.tgt_wcs, shape, interp)
    for tile in (5, 8):
        o2, f2 = dfr.reproject(src, c.src_wcs, c.tgt_wcs, shape, interp, tile=tile)
        assert torch.equal(o, o2) and torch.equal(f, f2), tile
    outs, fps = dfr.reproject_batch([src, src], [c.src_wcs] * 2, c.tgt_wcs, shape, interp)
    assert all(torch.equal(x, o) for x in outs) and all(torch.equal(x, f) for x in fps)


@pytest.mark.parametrize("interp", ["nearest", "bilinear"])
@pytest.mark.parametrize("rot", [2.0, 4.0, 45.0, 90.0, 178.0])
def test_rotated_maps_keep_their_bits(dfr, interp, rot):
    """Above the size line a turned map takes the square tile."""
    c = configs.sip3(scale=0.6)
    from synth import WcsParams
    tw = WcsParams.tan(c.tgt_wcs.crval, 2.85, rot, c.out_shape)
    src = torch.from_numpy(c.src).cuda()
    print(f"rotated interp={interp} rot={rot}", flush=True)
    o, f = dfr.reproject(src, c.src_wcs, tw, c.out_shape, interp)
    for tile in (5, 8):
        o2, f2 = dfr.reproject(src, c.src_wcs, tw, c.out_shape, interp, tile=tile)
        assert torch.equal(o, o2) and torch.equal(f, f2), tile
