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


def _kicked(precision, force, torque, mass):
    """Quotients force / mass and torque / (0.4 mass r r) as a DEM step takes
    them: 1,000 spheres at rest out of each other's reach, without gravity, the
    held fluid force, the stored torque and the mass put into a checkpoint.
    With a time step that is a power of two the step's two half kicks of equal
    size (one for the torque, whose new value is zero) scale them exactly."""
    torch = pytest.importorskip("torch")
    wl = synth.lattice(n_side=(10, 10, 10), spacing_factor=1.5)
    dt = 2.0 ** -17
    wl.dem.update(dt=dt, gravity=[0.0, 0.0, 0.0])
    wl.x[2] += 1e-3  # off the floor
    wl.v[:] = 0.0
    wl.w[:] = 0.0
    gb = gpu_bed(wl, precision)
    blob = gb.checkpoint().cpu()
    at, n = 256, wl.n
    for name, size in [("pr", 32), ("v", 24), ("w", 24), ("Fc", 24), ("Tc", 24), ("ffp", 24), ("rad", 8), ("mass", 8)]:
        new = {"Tc": torque, "ffp": force, "mass": mass}.get(name)
        if new is not None:
            blob[at:at + size * n] = torch.from_numpy(np.ascontiguousarray(new).view(np.uint8).reshape(-1))
        at = (at + size * n + 255) // 256 * 256
    gb.restore(blob)
    gb.step(1)
    st = gpu_state(gb)
    return st["v"] / dt, st["w"] / (0.5 * dt), 0.4 * mass * wl.radius * wl.radius, gb


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_infinite_quotients(precision):
    """An infinite torque gives an infinite spin, not a NaN (an infinite force
    puts its sphere at an infinite overlap with a wall within the step, which is
    a NaN by itself)."""
    for big in (np.inf, -np.inf):
        torque, mass = np.zeros((3, 1000)), np.full(1000, 3e-5)
        torque[2, 499] = big
        v, w, inertia, gb = _kicked(precision, np.zeros((3, 1000)), torque, mass)
        assert np.array_equal(w, torque / inertia)
        assert np.max(np.abs(v)) == 0.0
        assert gb.poll()[0] == 0


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_quotients_of_the_kicks(precision):
    """Newton steps against the division: the same bits over the exponent
    range, masses with every mantissa bit set among them; one unit in the last
    place where such a mass divides a power of two (the exception of a residual
    step after a reciprocal rounded to nearest)."""
    rng = np.random.default_rng(11)

    def numbers(lo, hi, size):
        return rng.choice([-1.0, 1.0], size) * rng.uniform(1.0, 2.0, size) * 2.0 ** rng.integers(lo, hi, size)

    ones = np.arange(1000) % 4 == 0
    mass = np.abs(numbers(-60, 20, 1000))
    mass[ones] = (2.0 - 2.0 ** -52) * 2.0 ** rng.integers(-60, 20, int(ones.sum()))
    force, torque = numbers(-400, -60, (3, 1000)), numbers(-400, 0, (3, 1000))  # no sphere reaches another
    force[0, ::3] = 0.0
    power = np.zeros((3, 1000), dtype=bool)
    power[2, ::8] = True
    force[2, ::8] = 2.0 ** rng.integers(-400, -60, 125)
    v, w, inertia, _ = _kicked(precision, force, torque, mass)
    assert np.array_equal(w, torque / inertia)
    want = force / mass
    assert np.array_equal(v[~power], want[~power])
    assert np.max(np.abs(v[power] / want[power] - 1.0)) <= 2.0 ** -52
