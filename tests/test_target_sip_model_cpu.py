"""The certificate of the cell models of a target with SIP, on the CPU: the
templates the device uses, compiled for the host (host_models.cpp), against the
oracle's FP64 chain at every pixel of sampled cells: the bound on the cubic, the
range that sizes a tile's source box, the distance from a rounding tie within
which nearest decides in FP64; distortions from ordinary to too strong for a
cubic, which must come back uncertified and still within their bound."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from synth import configs
from synth.sipfit import draw_sip
from tests.test_cell_model_cpu import (HALF, POWERS, cell_positions, model_fp32, model_positions,
                                       sample_cells)

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    import paper_2505_03932_amd as dfr
    from paper_2505_03932_amd import build
    so = str(tmp_path_factory.mktemp("models") / "libhost_models.so")
    flags = [f for f in build.CFLAGS if "offload-arch" not in f]
    subprocess.run([build._hipcc(), *flags, "--cuda-host-only", "-shared", "-o", so,
                    os.path.join(HERE, "host_models.cpp"), os.path.join(build.CSRC, "plan.cpp")],
                   check=True, capture_output=True)
    lib = C.CDLL(so)

    def model(sw, tw, cx, cy, any_order=True):
        s, t = dfr.api.CWcs(sw), dfr.api.CWcs(tw)
        mx, my, base = (C.c_double * 10)(), (C.c_double * 10)(), (C.c_int * 2)()
        rng, bound, tie = (C.c_double * 2)(), C.c_double(), C.c_double()
        cert = lib.host_cell_model(C.byref(s.s), C.byref(t.s), int(any_order), cx, cy, mx, my, base,
                                   rng, C.byref(bound), C.byref(tie))
        return {"coef_x": np.array(mx), "coef_y": np.array(my), "base": list(base),
                "range": np.array(rng), "bound": bound.value, "tie": tie.value, "certified": bool(cert)}
    return model


# (source frame, target order, factor on a distortion of about 1e-6 of the
# frame's side, whether every cell has to be certified)
CASES = [("plain", 2, 1.0, True), ("plain", 3, 50.0, True), ("sip3", 3, 1.0, True),
         ("sip3", 5, 20.0, False), ("sip3", 9, 20.0, False), ("grad", 3, 300.0, False),
         ("plain", 7, 3000.0, False), ("sip3", 4, 3000.0, False)]


@pytest.mark.parametrize("name,order,factor,all_certified", CASES)
def test_bounds_of_the_models(host, orc, name, order, factor, all_certified):
    c = {"plain": lambda: configs.plain(), "sip3": lambda: configs.sip3(),
         "grad": lambda: configs.grad(size=1024)}[name]()
    a, b = draw_sip(order, 0.5 * max(c.out_shape), np.random.default_rng(31))
    tw = c.tgt_wcs.copy(a=a * factor, b=b * factor)
    h = np.array([HALF ** (i + j) for i, j in POWERS])
    seen = 0
    for cx, cy in sample_cells(c.out_shape, 16, 5):
        m = host(c.src_wcs, tw, cx, cy)
        if order <= 5:  # zero coefficients above the order change nothing
            n = host(c.src_wcs, tw, cx, cy, any_order=False)
            assert all(np.array_equal(m[k], n[k]) for k in m)
        if all_certified:
            assert m["certified"], (cx, cy, m["bound"])
        if m["bound"] >= 1e29:
            assert not m["certified"] and m["tie"] == 0.5
            continue
        seen += 1
        pos, valid = cell_positions(orc, c.src_wcs, tw, cx, cy)
        assert valid.all()
        # (the oracle's chain and the composed map agree to about 1e-10 px)
        assert np.abs(model_positions(m) - pos).max() <= m["bound"] + 1e-8
        rnd = 2.0 ** -24 * (np.abs(m["coef_x"]) * h).sum() + 2.0 ** -24 * (np.abs(m["coef_y"]) * h).sum()
        if m["certified"]:
            assert m["bound"] <= 1e-6 + rnd * (1 + 1e-6) + 1e-9
        else:
            assert m["bound"] > 1e-6
        fp = model_fp32(m).astype(np.float64) + np.array(m["base"], np.float64)
        assert m["tie"] == 0.5 or np.abs(fp - pos).max() <= m["tie"] / 2 + 1e-9
        linear = dict(m, coef_x=np.where([i + j <= 1 for i, j in POWERS], m["coef_x"], 0.0),
                      coef_y=np.where([i + j <= 1 for i, j in POWERS], m["coef_y"], 0.0))
        beyond = np.abs(model_positions(linear) - pos).reshape(-1, 2).max(0)
        assert (beyond <= m["range"] + 1e-8).all(), (beyond, m["range"])
    assert seen > 0
