"""Neighbour lists and carried histories where a broad search can go wrong:
beds that rebuild their lists on almost every step, with list lengths that are
no multiple of a lane's share, particles away from their home cell, unsorted
beds, stencils cut off by every wall, and rolling friction; and the bed sizes at
which more lanes share a list."""
import numpy as np
import pytest

from paper_2211_01185_amd import cfddem, synth
from tests.parity_util import TOL, assert_close, compare_contacts, compare_states, gpu_bed, gpu_state, oracle_bed

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")

VARIANTS = [(p, lanes, mu_r) for p in ("fp64", "fp32") for lanes in (1, 2, 4) for mu_r in (0.0, 0.1)]


def _moving_lattice(n_side, mu_r):
    """Touching lattice in a box without clearance along x, in fast motion."""
    wl = synth.lattice(n_side=n_side)
    wl.v[:] = np.random.default_rng(3).normal(0.0, 0.3, wl.v.shape)
    wl.x[0] -= 0.005
    wl.dem["box_hi"][0] -= 0.01
    wl.dem["mu_r"] = mu_r
    return wl


@pytest.mark.parametrize("resort_every", [5, 1000])
@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_rebuilt_lists_against_the_oracle(lanes, resort_every):
    wl = _moving_lattice((9, 8, 11), 0.1)
    gb = gpu_bed(wl, "fp64", lanes=lanes, resort_every=resort_every, skin=1e-5)
    ob, _ = oracle_bed(wl)
    for _ in range(4):
        gb.step(3)
        ob.step(3)
        # up to twelve steps: a single step's tolerance for each
        assert compare_contacts(gb, ob, 12 * TOL["fp64"]) > 1500
        compare_states(gb, ob, 12 * TOL["fp64"], keys=("x", "v", "w", "Fc", "Tc"))
    assert gb.poll()[0] == 0


@pytest.mark.parametrize("precision,lanes,mu_r", VARIANTS)
def test_rebuilt_lists_have_the_same_bits_each_time(precision, lanes, mu_r):
    """Enough wavefronts to fill the chip; nothing may depend on their order."""
    wl = _moving_lattice((32, 32, 32), mu_r)
    runs = []
    for _ in range(2):
        gb = gpu_bed(wl, precision, lanes=lanes, resort_every=7, skin=1e-5)
        gb.step(20)
        runs.append((gpu_state(gb), gb.read_contacts()))
        assert gb.poll()[0] == 0
    (a, ca), (b, cb) = runs
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    for p, q in zip(ca, cb):
        assert np.array_equal(p, q)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [1, 8192, 8193, 40960, 40961])
def test_sizes_where_more_lanes_share_a_list(n, precision):
    """A single bed against a batch of one, which never shares a list's part."""
    wl = _moving_lattice((32, 32, 41) if n > 8193 else (16, 16, 33), 0.1)
    wl.x, wl.v, wl.w = wl.x[:, :n].copy(), wl.v[:, :n].copy(), wl.w[:, :n].copy()
    wl.radius, wl.density = wl.radius[:n].copy(), wl.density[:n].copy()
    single, other = gpu_bed(wl, precision, skin=1e-5), gpu_bed(wl, precision, skin=1e-5)
    batch = cfddem.Batch([other])
    single.step(3)
    batch.step(3)
    a, b = gpu_state(single), gpu_state(other)
    for k in ("x", "v", "w", "Fc", "Tc"):
        assert_close(k, a[k], b[k], 3 * TOL[precision])  # a single step's tolerance for each
    for p, q in zip(single.read_contacts()[:2], other.read_contacts()[:2]):
        assert np.array_equal(p, q)
    assert single.poll()[0] == 0 and other.poll()[0] == 0


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n_side", [(6, 6, 6), (21, 21, 20)])  # four and two lanes share a list's part
def test_full_lists_shared_by_more_lanes(n_side, precision):
    """Lists of the capacity's length, the last round of which leaves some of
    the sharing lanes past the list's end, from a capacity of one entry on."""
    wl = synth.lattice(n_side=n_side)
    for keep, longest in ((None, 6), (2, 1)):  # the whole lattice; two neighbours of it
        if keep:
            wl.x, wl.v, wl.w = wl.x[:, :keep].copy(), wl.v[:, :keep].copy(), wl.w[:, :keep].copy()
            wl.radius, wl.density = wl.radius[:keep].copy(), wl.density[:keep].copy()
        gb = gpu_bed(wl, precision, max_neighbors=longest)
        ob, _ = oracle_bed(wl)
        for steps in (0, 1, 2):
            gb.step(steps)
            ob.step(steps)
            tol = (1 + steps) * TOL[precision]  # a single step's tolerance for each
            compare_contacts(gb, ob, tol)
            compare_states(gb, ob, tol, keys=("x", "v", "w", "Fc", "Tc"))
        assert gb.poll()[0] == 0


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mu_r", [0.0, 0.1])
@pytest.mark.parametrize("n_side", [(12, 12, 28), (35, 35, 34)])  # four lanes to a list's part, and one
def test_every_share_of_a_list_has_the_same_bits_each_time(n_side, mu_r, precision):
    wl = _moving_lattice(n_side, mu_r)
    runs = []
    for _ in range(2):
        gb = gpu_bed(wl, precision, resort_every=7, skin=1e-5)
        gb.step(20)
        runs.append((gpu_state(gb), gb.read_contacts()))
        assert gb.poll()[0] == 0
    (a, ca), (b, cb) = runs
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    for p, q in zip(ca, cb):
        assert np.array_equal(p, q)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_batches_have_the_same_bits_each_time(lanes, precision):
    """A bed with rolling friction and one without (a kernel for each), large
    enough to fill the chip."""
    runs = []
    for _ in range(2):
        beds = [gpu_bed(_moving_lattice((32, 32, 32), mu_r), precision, lanes=lanes, resort_every=7, skin=1e-5)
                for mu_r in (0.0, 0.1)]
        batch = cfddem.Batch(beds)
        for _ in range(4):
            batch.step(5)
        runs.append([(gpu_state(b), b.read_contacts()) for b in beds])
        assert all(b.poll()[0] == 0 for b in beds)
        batch.close()
    for (a, ca), (b, cb) in zip(*runs):
        for k in a:
            assert np.array_equal(a[k], b[k]), k
        for p, q in zip(ca, cb):
            assert np.array_equal(p, q)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mu_r", [0.0, 0.1])
def test_a_part_of_a_list_has_the_same_sum_for_any_number_of_lanes(mu_r, precision):
    """The same touching spheres, alone (four lanes), and with others at rest
    beside them that make the bed large enough for two lanes and for one."""
    wl = _moving_lattice((12, 11, 13), mu_r)
    wl.dem["gravity"] = [0.0, 0.0, 0.0]
    n, d, top = wl.n, 2.0 * float(wl.radius[0]), float(wl.dem["box_hi"][2])
    wl.dem["box_hi"] = [0.15, 0.15, 0.25]
    wl.fluid["n_el"] = [10, 10, 16]
    k = np.arange(41000)
    rest = np.stack([(1 + k % 36) * 1.3 * d, (1 + k // 36 % 36) * 1.3 * d, top + (1 + k // 1296) * 1.3 * d])
    runs = []
    for extra in (0, 10000, 41000):
        one = synth.lattice(n_side=(2, 2, 2))
        one.dem, one.fluid = wl.dem, wl.fluid
        one.x = np.concatenate([wl.x, rest[:, :extra]], 1)
        one.v = np.concatenate([wl.v, np.zeros((3, extra))], 1)
        one.w = np.concatenate([wl.w, np.zeros((3, extra))], 1)
        one.radius, one.density = np.full(n + extra, 0.5 * d), np.full(n + extra, 2500.0)
        gb = gpu_bed(one, precision, skin=1e-5, resort_every=7)
        gb.step(10)
        assert gb.poll()[0] == 0
        st = {key: v[:, :n] for key, v in gpu_state(gb).items()}
        runs.append((st, gb.read_contacts()))
    for st, contacts in runs[1:]:
        for key in st:
            assert np.array_equal(st[key], runs[0][0][key]), key
        for p, q in zip(contacts, runs[0][1]):
            assert np.array_equal(p, q)
    assert len(runs[0][1][0]) > 2000


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mu_r", [0.0, 0.1])
@pytest.mark.parametrize("lanes", [1, 2, 4])
@pytest.mark.parametrize("n_side", [(16, 16, 20), (24, 24, 30), (36, 36, 36)])
def test_a_batch_of_one_has_the_bits_of_the_bed_alone(n_side, lanes, mu_r, precision):
    wl = _moving_lattice(n_side, mu_r)
    alone, other = (gpu_bed(wl, precision, lanes=lanes, resort_every=7, skin=1e-5) for _ in range(2))
    batch = cfddem.Batch([other])
    alone.step(10)
    batch.step(10)
    a, b = gpu_state(alone), gpu_state(other)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    for p, q in zip(alone.read_contacts(), other.read_contacts()):
        assert np.array_equal(p, q)
    assert alone.poll()[0] == 0 and other.poll()[0] == 0
    batch.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [6144, 6145])
def test_largest_bed_of_four_lanes_and_the_next(n, precision):
    """A bed's lanes change from four to two; a batch of one takes one."""
    wl = _moving_lattice((12, 16, 33), 0.1)
    wl.x, wl.v, wl.w = wl.x[:, :n].copy(), wl.v[:, :n].copy(), wl.w[:, :n].copy()
    wl.radius, wl.density = wl.radius[:n].copy(), wl.density[:n].copy()
    alone, other = (gpu_bed(wl, precision, skin=1e-5) for _ in range(2))
    batch = cfddem.Batch([other])
    alone.step(3)
    batch.step(3)
    a, b = gpu_state(alone), gpu_state(other)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    for p, q in zip(alone.read_contacts(), other.read_contacts()):
        assert np.array_equal(p, q)
    assert alone.poll()[0] == 0 and other.poll()[0] == 0
    batch.close()


@pytest.mark.parametrize("resort_every", [4, 1000])
@pytest.mark.parametrize("lanes", [1, 2, 4])
@pytest.mark.parametrize("n_el", [[10, 10, 10], [6, 9, 7]])  # cells of 1.06 d_max; of 1.8, 1.2 and 1.5
def test_no_partner_is_missed_among_spheres_of_many_sizes(n_el, lanes, resort_every):
    """Radii from 0.4 to 1.6 mm in a box away from the origin, in fast motion:
    the contacts at the bed's own positions, found by brute force, before and
    after broad searches that leave out the cells out of reach."""
    rng = np.random.default_rng(12)
    wl = synth.lattice(n_side=(2, 2, 2))
    lo = np.array([-0.7, 1.3, 20.0])
    k = np.arange(16 ** 3)
    x = 1.9e-3 * (np.stack([k % 16, k // 16 % 16, k // 256]) + 0.6) + rng.uniform(-4e-4, 4e-4, (3, k.size))
    wl.x = x + lo[:, None] + 1.5e-3  # away from the walls
    wl.radius = rng.uniform(0.4e-3, 1.2e-3, k.size)
    wl.radius[::40] = 1.6e-3
    wl.density = np.full(k.size, 2500.0)
    wl.v, wl.w = rng.normal(0.0, 0.5, x.shape), np.zeros(x.shape)
    wl.dem["box_lo"], wl.dem["box_hi"] = list(lo), list(lo + 0.0340)
    wl.dem.update(E=1e4, E_w=1e4)  # the overlaps come apart slowly
    wl.fluid["n_el"] = n_el
    gb = gpu_bed(wl, "fp64", lanes=lanes, resort_every=resort_every, skin=5e-5, cell_capacity=64, max_neighbors=64)
    found = 0
    for _ in range(12):
        gb.step(5)
        assert gb.poll()[0] == 0
        p = gb.read_state()["x"].cpu().numpy()
        d = p[:, None, :] - p[:, :, None]
        rs = wl.radius[:, None] + wl.radius[None, :]
        touch = rs * rs - (d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) > 0.0
        i, j, _ = gb.read_contacts()
        got = np.zeros_like(touch)
        got[i[j >= 0], j[j >= 0]] = True
        want = np.triu(touch, 1)
        assert np.array_equal(got, want)
        found += int(want.sum())
    assert found > 12 * 3000
