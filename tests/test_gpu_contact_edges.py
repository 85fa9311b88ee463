"""The contact law at the ends of its ranges against the oracle: overlaps from
1e-9 of the distance to a fifth of it, partners of very unequal size and mass,
forces whose squares underflow single precision, and coincident centres."""
import numpy as np
import pytest

from paper_2211_01185_amd import synth
from tests.parity_util import TOL, assert_close, gpu_bed, gpu_state, oracle_bed

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")


def _pair(overlap, ratio, density_ratio, spin):
    """Two spheres off every axis, overlapping by `overlap` of their distance."""
    wl = synth.plain(n=2)
    r = np.array([1.5e-3, 1.5e-3 * ratio])
    u = np.array([0.36, 0.48, 0.8])
    wl.radius[:] = r
    wl.density[:] = [2500.0, 2500.0 * density_ratio]
    wl.x[:, 0] = [0.02, 0.021, 0.1]
    wl.x[:, 1] = wl.x[:, 0] + u * (r.sum() / (1.0 + overlap))
    wl.v[:] = [[0.01, -0.02], [0.0, 0.01], [0.003, -0.001]]
    wl.w[:] = [[30.0, -10.0], [-20.0, 5.0], [4.0, 40.0]]
    if not spin:  # at rest: the spring alone
        wl.w[:] = 0.0
        wl.v[:] = 0.0
    return wl


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("ratio,density_ratio", [(1.0, 1.0), (0.25, 1e-6), (0.25, 1e6)])
@pytest.mark.parametrize("overlap", [1e-9, 1e-4, 0.2])
def test_overlap_and_size_ratios(overlap, ratio, density_ratio, precision):
    wl = _pair(overlap, ratio, density_ratio, True)
    gb = gpu_bed(wl, precision)
    ob, _ = oracle_bed(wl)
    # the overlap is a difference: a last-bit error of the distance is 2^-52 /
    # overlap of it, and the force goes with its 3/2 power
    tol = TOL[precision] + 4.0 * 2.0 ** -52 / overlap
    for steps in (0, 1):
        gb.step(steps)
        ob.step(steps)
        g, o = gpu_state(gb), ob.state()
        assert_close("Fc", g["Fc"], o["Fc"], tol)
        assert_close("Tc", g["Tc"], o["Tc"], tol)
        assert_close("v", g["v"], o["v"], tol)


def test_forces_that_underflow_single_precision_when_squared():
    wl = _pair(1e-6, 1.0, 1.0, False)
    wl.dem.update(E=1e-9, E_w=1e-9)
    gb = gpu_bed(wl, "fp32")
    ob, _ = oracle_bed(wl)
    g, o = gpu_state(gb), ob.state()
    assert 0.0 < np.max(np.abs(o["Fc"])) < 1e-20
    assert_close("Fc", g["Fc"], o["Fc"], TOL["fp32"] + 4.0 * 2.0 ** -52 / 1e-6)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_coincident_centres_are_an_error(precision):
    from paper_2211_01185_amd import cfddem

    wl = _pair(0.2, 1.0, 1.0, True)
    wl.x[:, 1] = wl.x[:, 0]
    gb = gpu_bed(wl, precision)
    gb.step(1)
    err, _ = gb.poll()
    assert err == cfddem.DEM_E_NAN
