"""What the library asks of the HIP runtime, call by call, with a recording
stand-in for the runtime (fake_hip.cpp): no GPU, no kernel runs.  Calls under
stream capture, allocation failures and failed launches are forced from here.

Each case runs in a process of its own: the stand-in has to be loaded before
libdfr.so, and torch (whose own HIP runtime would be found first) not at all."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, importlib.util, math, os, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.fake_log.restype = C.c_char_p
sys.modules["torch"] = None
spec = importlib.util.spec_from_file_location("_lib", sys.argv[2])
lib = importlib.util.module_from_spec(spec)
spec.loader.exec_module(lib)
fake.fake_set_library(lib.LIB_PATH.encode())

keep = []

def wcs(rot=0.0, ab=0, apbp=0, size=64, eps=1e-7):
    w = lib.dfr_wcs()
    w.crpix[:] = [0.5 * (size + 1)] * 2
    w.crval[:] = [150.0, 2.0]
    s, r = 8e-4, math.radians(rot)
    w.cd[:] = [-s * math.cos(r), s * math.sin(r), s * math.sin(r), s * math.cos(r)]
    for order, names in ((ab, "ab"), (apbp, ("ap", "bp"))):
        for n in names if order else ():
            c = (C.c_double * (order + 1) ** 2)()
            c[2] = eps  # the (0, 2) term
            keep.append(c)
            setattr(w, n + "_order", order)
            setattr(w, n, C.addressof(c))
    return w

def opts():
    o = lib.dfr_options()
    lib.dfr_options_init(o)
    return o

def names():
    return [n.decode() for n in fake.fake_log().split()]

IMG = 1 << 20  # an address: no kernel runs, nothing reads it
STREAM = 4096

def reproject(n=64, out=64, ab=0, apbp=2, rot=0.3):
    return lib.dfr_reproject(IMG, n, n, n, wcs(rot, 0, apbp, n), wcs(0.0, ab, 0, out), out, out, 1,
                             IMG, IMG, opts(), STREAM)

def frames(k, n=64, apbp=2):
    f = (lib.dfr_frame * k)()
    for i in range(k):
        f[i].src, f[i].h, f[i].w, f[i].pitch, f[i].wcs = IMG, n, n, n, wcs(0.3, 0, apbp, n)
    return f

def pointers(k):
    return (C.c_void_p * k)(*[IMG] * k)

def stack(kind, k=3, out=64, ab=0):
    tw = wcs(0.0, ab, 0, out)
    if kind == "batch":
        return lib.dfr_reproject_batch(k, frames(k), tw, out, out, 1, pointers(k), None, opts(), STREAM)
    if kind == "coadd":
        return lib.dfr_coadd_batch(k, frames(k), tw, out, out, 1, IMG, IMG, None, 0, opts(), STREAM)
    boxes = (C.c_int32 * (4 * k))(*[0, 0, out, out] * k)
    if kind == "boxes":
        return lib.dfr_batch_boxes(k, frames(k), tw, out, out, 1, opts(), STREAM,
                                   C.cast(boxes, C.c_void_p))
    return lib.dfr_reproject_batch_cropped(k, frames(k), tw, out, out, 1,
                                           C.cast(boxes, C.c_void_p), pointers(k), None, opts(), STREAM)

OK, DEVICE, NOMEM = 0, 5, 6
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "fake_hip.cpp")], check=True)
    return so


def run(fake, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, fake,
                        os.path.join(ROOT, "paper_2505_03932_amd", "_lib.py")],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_the_stand_in_is_the_one_bound(fake):
    run(fake, """
assert reproject() == OK
assert len(names()) == 1 and "reproject_small" in names()[0], names()
assert reproject(out=2048) == OK
assert "cell_models_kernel" in names()[1] and "reproject_tiles" in names()[2], names()
""")


@pytest.mark.parametrize("kind", ["batch", "coadd", "boxes", "cropped"])
def test_stack_calls_are_refused_under_capture(fake, kind):
    """Their frame table is copied from a staging buffer that later calls
    refill, and a graph launched into a capturing stream runs at once, with
    whatever table an earlier call left: refused before anything is queued,
    and the stream's later calls work."""
    run(fake, f'''
for _ in range(5):
    assert stack({kind!r}) == OK
fake.fake_set_capturing(1)
before = (fake.fake_copies(), fake.fake_graph_launches(), len(names()))
for _ in range(5):
    assert stack({kind!r}) == DEVICE
assert before == (fake.fake_copies(), fake.fake_graph_launches(), len(names()))
assert fake.fake_last_error() == 0
fake.fake_set_capturing(0)
for _ in range(5):
    assert stack({kind!r}) == OK
''')


def test_captured_target_with_sip_keeps_no_scratch(fake):
    """Whatever the stream's workspace already holds, a captured call of a
    target with SIP records the tile kernel alone, on the anchored chain: no
    table whose address the graph would keep."""
    run(fake, '''
for out in (64, 2048):
    assert reproject(out=out, ab=2) == OK  # the stream's workspace exists now
    assert "cell_models_kernel" in names()[-2] and "reproject_tiles" in names()[-1], names()
    fake.fake_set_capturing(1)
    n = len(names())
    assert reproject(out=out, ab=2) == OK
    assert len(names()) == n + 1 and "reproject_tiles" in names()[-1], names()
    fake.fake_set_capturing(0)
''')


def plan(ab):
    return f"""
def plan(out=64):
    return lib.dfr_plan_create(64, 64, wcs(0.3, 0, 2), wcs(0.0, {ab}, 0, out), out, out, 1, opts(), STREAM)
"""


def test_plan_of_a_target_with_sip_created_under_capture(fake):
    """Such a plan needs no memory of its own (the anchored chain): none is
    asked for, which would end the capture, and no model kernel is recorded,
    which would leave the plan without models until a replay."""
    run(fake, plan(ab=2) + '''
fake.fake_set_capturing(1)
s, h = plan()
assert s == OK and names() == [] and fake.fake_mallocs() == 0 and fake.fake_last_error() == 0
assert lib.dfr_plan_execute(h, IMG, 64, IMG, None, STREAM) == OK
assert len(names()) == 1 and "reproject_tiles" in names()[0], names()
fake.fake_set_capturing(0)
assert lib.dfr_plan_destroy(h) == OK
s, h = plan()
assert s == OK and "cell_models_kernel" in names()[1] and fake.fake_mallocs() == 1
assert lib.dfr_plan_destroy(h) == OK
''')


@pytest.mark.parametrize("kind", ["single", "batch", "coadd"])
def test_target_with_sip_without_memory_for_models(fake, kind):
    """No memory for the table: the anchored chain runs, and the runtime's
    out-of-memory error, which the next check of a launch would take for its
    own, is not left behind."""
    run(fake, f'''
call = lambda ab=2: reproject(out=2048, ab=ab) if {kind!r} == "single" else stack({kind!r}, out=2048, ab=ab)
fake.fake_fail_malloc(1)
assert call() == OK
assert not any("cell_models" in n for n in names()), names()
assert fake.fake_last_error() == 0
fake.fake_fail_malloc(1)
assert lib.dfr_release() == OK
assert call(ab=0) == NOMEM  # a target without SIP has no other form
assert fake.fake_last_error() == 0 and call(ab=0) == OK
''')


@pytest.mark.parametrize("call", ["reproject()", "reproject(out=2048)", "reproject(out=2048, ab=2)",
                                  "stack('boxes')", "stack('cropped')", "backward()"])
@pytest.mark.parametrize("launch", [0, 1, 2])
def test_a_failed_launch_fails_its_own_call_only(fake, call, launch):
    """Whichever of a call's launches fails, the call says so and the next
    check of a launch, this library's or another's, does not find it again."""
    run(fake, f'''
def backward():
    return lib.dfr_reproject_backward(IMG, 64, 64, 64, wcs(0.3, 0, 2), wcs(), 64, 64, 1, IMG, IMG, IMG,
                                      opts(), STREAM)
assert {call} == OK
before = len(names())
assert {call} == OK
if len(names()) - before > {launch}:
    fake.fake_skip_launches({launch})
    fake.fake_fail_launch(1)
    assert {call} == DEVICE
    assert fake.fake_last_error() == 0
    assert {call} == OK
''')


def test_staging_is_allocated_once_a_size(fake):
    """Pinned memory is asked for by the first stack call on a stream and by
    the first larger one, not by the calls that follow."""
    run(fake, '''
asked = []
for k in [3] * 6 + [40] * 6 + [3] * 3 + [40]:
    assert stack("coadd", k) == OK
    asked.append(fake.fake_host_mallocs())
assert asked == [1] * 6 + [2] * 10, asked
''')


def test_new_geometry_estimates_each_tile_once(fake):
    """The set-up of a geometry not met before asks for the LDS of up to three
    tile shapes, each estimated once, whichever default tile applies; a stack
    adds one estimate per further frame."""
    run(fake, '''
def estimates(f):
    before = fake.fake_estimates()
    assert f() == OK
    return fake.fake_estimates() - before
counts = {}
for interp in (0, 1, 2):
    for out in (64, 2048, 4000, 6001):
        for rot in (0.1, 5.0, 45.0, 90.0):
            one = lambda: lib.dfr_reproject(IMG, 64, 64, 64, wcs(rot, 0, 2), wcs(0.0, 0, 0, out), out, out,
                                            interp, IMG, IMG, opts(), STREAM)
            counts[interp, out, rot] = estimates(one)
            assert estimates(one) == 0
print(counts)
assert all(1 <= c <= 3 for c in counts.values())
assert estimates(lambda: stack("batch", 3, out=6001)) <= 3 + 2
assert estimates(lambda: stack("coadd", 3)) == 3
''')


@pytest.mark.parametrize("order,most", [(0, 768), (3, 768), (4, 768), (5, 512)])
def test_one_launch_form_up_to_the_groups_that_run_at_once(fake, order, most):
    run(fake, f'''
def launched(rows):
    s = lib.dfr_reproject(IMG, 64, 64, 64, wcs(0.3, 0, {order}), wcs(), 32 * rows, 32, 1, IMG, IMG, opts(), STREAM)
    assert s == OK
    return names()[-1]
assert "reproject_small" in launched({most}) and "reproject_small" not in launched({most} + 1)
''')


def test_prepass_of_many_cells_takes_several_launches(fake):
    """A launch has fewer than 2^32 threads; the prepass rounds a strip one cell
    high up to blocks of 8x8 cells, so 2100 frames on one of 262144 cells reach
    that long before the memory of their models ends."""
    run(fake, '''
def coadd(k):
    return lib.dfr_coadd_batch(k, frames(k), wcs(), 32, 1 << 23, 1, IMG, IMG, None, 0, opts(), STREAM)
assert coadd(2000) == OK
assert ["cell_models_batch" in n for n in names()].count(True) == 1
assert coadd(2100) == OK
assert ["cell_models_batch" in n for n in names()].count(True) == 3
''')
