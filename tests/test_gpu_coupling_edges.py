"""Coupling steps at the mesh sizes where the classification pass comes in
(1,024 blocks of elements) and mostly empty meshes, against the oracle."""
import numpy as np
import pytest

from paper_2211_01185_amd import synth
from tests.parity_util import TOL, assert_close, gpu_bed, gpu_state, oracle_bed

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,elem_threads,n_el", [
    (1, 128, [1, 1, 1]), (300, 128, [16, 8, 8]), (300, 128, [5, 5, 41]), (300, 64, [16, 8, 8]), (300, 64, [5, 5, 41]),
    (300, 32, [16, 16, 8]), (300, 32, [5, 10, 41]), (300, 16, [16, 16, 16]), (300, 16, [10, 10, 41])])
def test_meshes_with_and_without_classification(n, elem_threads, n_el, precision):
    wl = synth.plain(n=n)
    lo, hi = wl.dem["box_lo"], wl.dem["box_hi"]
    wl.fluid["n_el"] = n_el
    nodes = synth.node_grid(lo, hi, n_el, 2)
    wl.U = np.stack([0.1 * nodes[1], 0.0 * nodes[0], 0.5 + nodes[2]])
    wl.P = 100.0 * (1.0 - synth.node_grid(lo, hi, n_el, 1)[2] / hi[2])
    gb = gpu_bed(wl, precision, elem_threads=elem_threads)
    ob, fl = oracle_bed(wl)
    U, P = (torch.as_tensor(f, dtype=torch.float64, device="cuda").contiguous() for f in (wl.U, wl.P))
    tol = TOL[precision]
    for step in range(3):  # a single step's tolerance for each
        out, ref = gb.couple(U, P, elem_sums=True), ob.couple(fl, wl.U, wl.P)
        assert np.array_equal(out["elem_sums"][0].cpu().numpy(), ref["elem_sums"][0])
        assert_close("eps_q", out["eps_q"].cpu().numpy(), ref["eps_q"], 1e-12 * (1 + step))
        for k in ("beta_q", "fpf_q"):
            assert_close(k, out[k].cpu().numpy(), ref[k], tol * (1 + step))
        assert_close("f_fp", gpu_state(gb)["ffp"], ob.state()["ffp"], tol * (1 + step))
        gb.step(1)
        ob.step(1)
    assert gb.poll()[0] == 0


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("elem_threads", [32, 64, 128])
@pytest.mark.parametrize("nz", [30, 34])
def test_elements_of_few_particles_beside_crowded_ones(nz, elem_threads, precision):
    """Q1 meshes of 1,920 and 2,176 elements with one particle each, some with
    none, 15, 16, 17, 18 and 100: the few-particle groups' bounds."""
    wl = synth.plain(n=2)
    n_el, hi = [8, 8, nz], np.array(wl.dem["box_hi"])
    h = hi / n_el
    e = np.arange(64 * nz)
    count = np.ones(e.size, dtype=int)
    count[[0, 7, 70, 500, 501, 900, 1300, 64 * nz - 1]] = [17, 16, 18, 0, 100, 15, 17, 16]
    rng = np.random.default_rng(5)
    x = []
    for i in e:
        base = np.array([i % 8, (i // 8) % 8, i // 64])
        k = rng.permutation(125)[:count[i]]
        cell = (np.stack([k % 5, (k // 5) % 5, k // 25], 1) + rng.uniform(0.4, 0.6, (k.size, 3))) / 5
        x.append((base + cell) * h)
    x = np.concatenate(x)[rng.permutation(count.sum())]
    wl.x = np.ascontiguousarray(x.T)
    n = wl.x.shape[1]
    wl.v, wl.w = rng.normal(0.0, 0.1, (3, n)), np.zeros((3, n))
    wl.radius, wl.density = np.full(n, 0.4e-3), np.full(n, 2500.0)
    wl.fluid.update(order=1, n_el=n_el)
    nodes = synth.node_grid(wl.dem["box_lo"], hi, n_el, 1)
    wl.U = np.stack([0.1 * nodes[1], 0.0 * nodes[0], 0.5 + nodes[2]])
    wl.P = 100.0 * (1.0 - nodes[2] / hi[2])
    gb = gpu_bed(wl, precision, elem_threads=elem_threads)
    ob, fl = oracle_bed(wl)
    U, P = (torch.as_tensor(f, dtype=torch.float64, device="cuda").contiguous() for f in (wl.U, wl.P))
    for _ in range(2):
        out, ref = gb.couple(U, P, elem_sums=True), ob.couple(fl, wl.U, wl.P)
        assert np.array_equal(out["elem_sums"][0].cpu().numpy(), ref["elem_sums"][0])
        assert_close("eps_q", out["eps_q"].cpu().numpy(), ref["eps_q"], 1e-12)
        for k in ("beta_q", "fpf_q"):
            assert_close(k, out[k].cpu().numpy(), ref[k], TOL[precision])
        assert_close("f_fp", gpu_state(gb)["ffp"], ob.state()["ffp"], TOL[precision])
    assert gb.poll()[0] == 0


def _mesh_of_counts(n_el, count, radius):
    """A Q1 bed whose elements hold the given numbers of particles (at most
    125), in random order, and its oracle's fields."""
    wl = synth.plain(n=2)
    hi = np.array(wl.dem["box_hi"])
    rng = np.random.default_rng(6)
    e = np.repeat(np.arange(count.size), count)
    k = np.concatenate([rng.permutation(125)[:c] for c in count])
    base = np.stack([e % n_el[0], (e // n_el[0]) % n_el[1], e // (n_el[0] * n_el[1])], 1)
    x = base + (np.stack([k % 5, (k // 5) % 5, k // 25], 1) + rng.uniform(0.4, 0.6, (k.size, 3))) / 5
    wl.x = np.ascontiguousarray((x * hi / n_el)[rng.permutation(k.size)].T)
    n = wl.x.shape[1]
    wl.v, wl.w = rng.normal(0.0, 0.1, (3, n)), np.zeros((3, n))
    wl.radius, wl.density = np.full(n, radius), np.full(n, 2500.0)
    wl.fluid.update(order=1, n_el=n_el)
    nodes = synth.node_grid(wl.dem["box_lo"], hi, n_el, 1)
    wl.U = np.stack([0.1 * nodes[1], 3.0 * nodes[0] * nodes[2], 0.5 + nodes[2] + 20.0 * nodes[0] * nodes[1]])
    wl.P = 100.0 * (1.0 - nodes[2] / hi[2])
    return wl


def _couple_against_the_oracle(wl, precision, elem_threads):
    """One coupling call against the oracle, and the call repeated to the bit."""
    gb = gpu_bed(wl, precision, elem_threads=elem_threads)
    ob, fl = oracle_bed(wl)
    U, P = (torch.as_tensor(f, dtype=torch.float64, device="cuda").contiguous() for f in (wl.U, wl.P))
    ref, tol = ob.couple(fl, wl.U, wl.P, smooth_L2=wl.fluid.get("smooth_L2")), TOL[precision]
    runs = []
    for _ in range(3):
        out = gb.couple(U, P, elem_sums=True)
        runs.append({**out, "ffp": gb.read_state()["ffp"].clone()})
    out = runs[0]
    assert np.array_equal(out["elem_sums"][0].cpu().numpy(), ref["elem_sums"][0])
    assert_close("eps_q", out["eps_q"].cpu().numpy(), ref["eps_q"], 1e-10 if wl.fluid.get("smooth_L2") else 1e-12)
    for k in ("beta_q", "fpf_q", "elem_sums"):
        assert_close(k, out[k].cpu().numpy(), ref[k], tol)
    assert_close("f_fp", out["ffp"].cpu().numpy(), ob.state()["ffp"], tol)
    for other in runs[1:]:
        for k in out:
            assert torch.equal(out[k], other[k]), k
    assert gb.poll()[0] == 0


LAWS = [dict(), dict(drag="gidaspow", model=1), dict(drag="koch_hill", beta_over_eps=1), dict(shear=1, model=1),
        dict(smooth_L2=5 * 0.8e-3 ** 2)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("elem_threads", [64, 128])
@pytest.mark.parametrize("law", range(len(LAWS)))
@pytest.mark.parametrize("n_el,radius", [
    ([8, 8, 34], 0.7e-3),   # 48 cells per element, groups for 2,168 elements
    ([8, 8, 34], 0.2e-3),   # 2,548 cells per element: a block for each
    ([8, 8, 30], 0.4e-3),   # 294 cells per element, 1,912 elements of few particles: a block for each
    ([8, 8, 30], 0.7e-3),   # 48 cells per element: without the split
    ([10, 10, 10], 0.7e-3)])  # without a list
def test_element_routes_of_every_law(n_el, radius, law, elem_threads, precision):
    count = np.ones(n_el[0] * n_el[1] * n_el[2], dtype=int)
    count[[0, 7, 70, 500, 501, 900, 960, count.size - 1]] = [17, 16, 18, 0, 100, 15, 17, 16]
    wl = _mesh_of_counts(n_el, count, radius)
    wl.fluid.update(LAWS[law])
    _couple_against_the_oracle(wl, precision, elem_threads)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("elem_threads", [64, 128])
def test_more_elements_of_either_kind_than_the_grid_takes_at_once(elem_threads, precision):
    """4,200 crowded elements (4,096 blocks) and 37,272 of one particle (8 x
    4,096 groups)."""
    count = np.ones(36 * 36 * 32, dtype=int)
    count[np.random.default_rng(7).permutation(count.size)[:4200]] = 17
    _couple_against_the_oracle(_mesh_of_counts([36, 36, 32], count, 0.1e-3), precision, elem_threads)


@pytest.mark.parametrize("elem_threads", [64, 128])
def test_crowded_meshes_without_the_split(elem_threads):
    """A mean of 17 particles in elements of few cells."""
    _couple_against_the_oracle(_mesh_of_counts([8, 8, 34], np.full(8 * 8 * 34, 17), 0.7e-3), "fp64", elem_threads)
