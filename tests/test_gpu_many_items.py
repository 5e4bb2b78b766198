"""A stack of more (frame, tile) items than one launch of a batch kernel takes
(2^23): several launches, the dense batch without its graph.  Frames on a strip
one cell high, so that the items are many and the images small; two sources in
turn, every frame bit for bit the single call's."""
import pytest
import torch

from synth import configs

pytestmark = pytest.mark.gpu
LIMIT = 1 << 23
H, W, TILE = 32, 65536, 1  # 2048 tiles of 32x32 a frame
N = LIMIT // 2048 + 37     # a whole round over the XCDs and a part of one in the last launch


@pytest.fixture(scope="module")
def dfr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_03932_amd as d
    yield d
    d.release()
    torch.cuda.empty_cache()


def _strip():
    c = configs.plain(size=64)
    one = torch.from_numpy(c.src).cuda()
    tw = c.tgt_wcs.copy(crpix=(c.tgt_wcs.crpix[0] + 30000.0, c.tgt_wcs.crpix[1] - 12.0))
    return [one, one.flip(0).contiguous()], [c.src_wcs, c.src_wcs], tw


def test_cropped(dfr):
    srcs, wcss, tw = _strip()
    want = [dfr.reproject(s, w, tw, (H, W), "bilinear")[0] for s, w in zip(srcs, wcss)]
    assert all(o.any() for o in want)
    boxes = [[0, i % H, W, 1] for i in range(N)]
    print(f"cropped stack of {N * 2048} items", flush=True)
    outs, _, _ = dfr.reproject_batch_cropped([srcs[i & 1] for i in range(N)],
                                             [wcss[i & 1] for i in range(N)], tw, (H, W), "bilinear",
                                             boxes=boxes, footprint=False, tile=TILE)
    wrong = torch.zeros((), device="cuda", dtype=torch.int64)
    for i, o in enumerate(outs):
        wrong += (o[0] != want[i & 1][i % H]).sum()
    assert int(wrong) == 0


def test_dense(dfr):
    srcs, wcss, tw = _strip()
    want = [dfr.reproject(s, w, tw, (H, W), "bilinear")[0] for s, w in zip(srcs, wcss)]
    out = torch.full((N, H, W), -7.0, device="cuda")  # 35 GB
    print(f"dense stack of {N * 2048} items", flush=True)
    dfr.reproject_batch([srcs[i & 1] for i in range(N)], [wcss[i & 1] for i in range(N)], tw, (H, W),
                        "bilinear", outs=list(out.unbind(0)), footprint=False, tile=TILE)
    for k in (0, 1):
        for part in out[k::2].split(256):
            assert torch.equal(part, want[k].expand_as(part))
