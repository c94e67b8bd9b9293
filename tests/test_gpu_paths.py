"""The recorded paths at the edges of their layout: packets that are not full,
segments that end by slots, visits or hits, rays without hits, shifted images,
and packets split into parts."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _case(which):
    """A workload and the leaf size of its tree."""
    if which == "one":                       # one particle: one ray to a packet
        return W.isothermal_halo(n=1, n_bins=1, seed=3), 0
    if which == "packet_less_one":
        return W.isothermal_halo(n=63, n_bins=1, seed=4), 0
    if which == "packet":
        return W.isothermal_halo(n=64, n_bins=1, seed=5), 0
    if which == "packet_plus_one":
        return W.isothermal_halo(n=65, n_bins=1, seed=6), 0
    if which == "visits":                    # one-particle leaves: 128 visits a segment
        return W.isothermal_halo(n=700, n_bins=1, seed=7), 1
    if which == "slots":                     # many leaves, few rays in each: 1024 slots
        wl = W.isothermal_halo(n=6000, n_bins=1, seed=8)
        wl.h = (wl.h * 0.35).astype(np.float32)
        return wl, 16
    if which == "no_hits":                   # kernels that hold their own particle only
        wl = W.isothermal_halo(n=300, n_bins=1, seed=9)
        wl.h = (wl.h * 1e-3).astype(np.float32)
        return wl, 0
    if which == "images":                    # every ray crosses the box several times
        return W.uniform_lattice(n_side_lattice=7, box=20.0, l_ray=67.0), 0
    return W.lognormal_field(n_grid=20, box=1562.5, n_bins=1, n_side=2), 0   # parts = 1


CASES = ["one", "packet_less_one", "packet", "packet_plus_one", "visits", "slots", "no_hits",
         "images", "field"]


@pytest.mark.parametrize("near_far", [0, 1])
@pytest.mark.parametrize("which", CASES)
def test_recorded_paths_hold_the_walk(which, near_far):
    """Columns over the recorded paths against the traversal's: the same FP32
    products, summed in FP64 in another order, so a ray's columns differ by at
    most its intersections times 2^-53 of their (positive) sum, 1e-11 for any
    ray here.  The paths by rows against the walk's hit lists: the same
    particles in the same order, the same factors.  A second recording gives
    the same columns bit for bit."""
    from paper_1304_4235_amd import Solver
    wl, leaf = _case(which)
    rng = np.random.default_rng(1)
    x = torch.tensor(rng.uniform(1e-6, 1.0, wl.n))
    src = np.sort(rng.choice(wl.n, min(wl.n, 130), replace=False))
    out = []
    for paths in (1, 0):
        s = Solver.from_workload(wl, leaf_size=leaf, record_paths=paths, build=False)
        s.set_scheme(near_far)
        s.build_tree()
        s.set_state(x)
        N, hits = s.compute_columns()
        near = s.near_columns().cpu().numpy() if near_far else None
        out.append((N.cpu().numpy(), hits, near))
        if paths:
            off, j, fac = s.path_rows(src)
            ho, hj, _, hf = s.hits_rows(src)
            np.testing.assert_array_equal(off, ho)
            np.testing.assert_array_equal(j, hj)
            np.testing.assert_array_equal(fac, hf)
            s.build_tree()                               # one walk, sized from the first
            s.set_state(x)
            again, _ = s.compute_columns()
            np.testing.assert_array_equal(again.cpu().numpy(), out[0][0])
        s.close()
    (N1, h1, n1), (N0, h0, n0) = out
    assert h1 == h0
    np.testing.assert_allclose(N1, N0, rtol=1e-11, atol=0)
    if near_far:
        np.testing.assert_allclose(n1, n0, rtol=1e-11, atol=0)


def test_row_products_of_the_recorded_paths():
    """What takes the paths by rows: the density order's blocks (paths expanded
    into rows) against the same blocks without recorded paths, and the
    transposed product with one atomic add per intersection against the gather
    over transposed paths, on a tree whose packets are not full."""
    from paper_1304_4235_amd import Solver
    wl = W.isothermal_halo(n=3001, n_bins=8, seed=12)
    xs = []
    for paths in (1, 0):
        s = Solver.from_workload(wl, record_paths=paths)
        s.set_update_rule(n_blocks=7)
        xs.append(s.iterate(3, 0.0)["x"].cpu().numpy())
        s.close()
    np.testing.assert_allclose(xs[0], xs[1], rtol=1e-9)
    s = Solver.from_workload(wl, record_paths=1)
    g = torch.ones(wl.n, dtype=torch.float64, device="cuda")
    dn = []
    for mode in (0, 1):
        s.set_tuning(adjoint_scatter=mode)
        s.forward(3)
        dn.append(s.backward(g, None)[1].cpu().numpy())
    np.testing.assert_allclose(dn[1], dn[0], rtol=1e-9, atol=1e-12 * np.abs(dn[0]).max())
    s.close()


@pytest.mark.parametrize("which", ["one", "packet_plus_one", "slots", "images", "field"])
def test_recording_in_pieces(which):
    """The least path buffer that rrt_count_paths names holds no whole log: the
    paths are recorded a range of units at a time, to the same columns bit for
    bit; half of it is refused."""
    from paper_1304_4235_amd import RRTError, Solver
    wl, leaf = _case(which)
    x = torch.tensor(np.random.default_rng(2).uniform(1e-6, 1.0, wl.n))
    s = Solver.from_workload(wl, leaf_size=leaf, record_paths=1)
    need = s.count_paths()
    s.set_state(x)
    N, hits = s.compute_columns()
    N = N.clone()
    assert need["bytes_paths"] < need["bytes_one_walk"]
    t = Solver.from_workload(wl, leaf_size=leaf, record_paths=1, path_budget=need["bytes_paths"])
    for _ in range(2):
        t.build_tree()
        t.set_state(x)
        got, h = t.compute_columns()
        assert h == hits == t.timing()["path_hits"]
        assert torch.equal(got, N)
    u = Solver.from_workload(wl, leaf_size=leaf, record_paths=1,
                             path_budget=need["bytes_paths"] // 2)
    u.set_state(x)
    with pytest.raises(RRTError, match="RRT_E_WORKSPACE"):
        u.compute_columns()
    for q in (s, t, u):
        q.close()


def test_paths_over_many_images():
    """Images that a ray reaches up to 9000 box lengths away: columns over the
    recorded paths against the traversal's (FP64 sums in another order)."""
    from paper_1304_4235_amd import Solver
    out = []
    for paths in (1, 0):
        s = Solver(l_ray=9000.0, box=1.0, record_paths=paths)
        s.set_particles(np.array([[0.5, 0.5, 0.5]], np.float32), np.array([0.3], np.float32),
                        np.array([1e15], np.float32), np.array([1e-2], np.float32),
                        np.array([1e4], np.float32))
        s.set_rays(np.array([[1.0, 0.0, 0.0]]))
        s.set_spectrum(np.array([6e-18]), np.array([1e5]))
        s.build_tree()
        N, hits = s.compute_columns()
        out.append((N.cpu().numpy(), hits))
        s.close()
    assert out[0][1] == out[1][1] >= 9000
    np.testing.assert_allclose(out[0][0], out[1][0], rtol=1e-11)


@pytest.mark.parametrize("l_ray,n_ray", [(9000.0, 6), (60000.0, 1)])
def test_least_buffer_holds_a_lone_rays_many_visits(l_ray, n_ray):
    """One ray to a packet and one pair to a visit, thousands of visits: a
    segment ends by its slots, visits or hits as everywhere else, so the least
    buffer that rrt_count_paths names holds the paths here too, to the columns
    of the full buffer bit for bit."""
    from paper_1304_4235_amd import Solver
    axes = np.concatenate([np.eye(3), -np.eye(3)])       # a ray meets one line of images
    out, need = [], None
    for budget in (0, 1):
        s = Solver(l_ray=l_ray, box=1.0, record_paths=1,
                   path_budget=need["bytes_paths"] if budget else 0)
        s.set_particles(np.array([[0.5, 0.5, 0.5]], np.float32), np.array([0.3], np.float32),
                        np.array([1e15], np.float32), np.array([1e-2], np.float32),
                        np.array([1e4], np.float32))
        s.set_rays(axes[:n_ray])
        s.set_spectrum(np.array([6e-18]), np.array([1e5]))
        s.build_tree()
        need = s.count_paths()
        N, hits = s.compute_columns()
        assert hits == need["hits"] == s.timing()["path_hits"]
        out.append(N.cpu().numpy())
        s.close()
    np.testing.assert_array_equal(out[0], out[1])


def _tile_case(which):
    if which == "long":                      # over 2000 hits a ray: 16 rows to a tile
        return W.uniform_lattice(n_side_lattice=5, box=20.0, l_ray=700.0), 0
    if which == "mid":                       # a packet in two tiles of 32 rows
        return W.uniform_lattice(n_side_lattice=5, box=20.0, l_ray=300.0), 0
    return _case(which)


@pytest.mark.parametrize("which", ["one", "packet_less_one", "packet", "packet_plus_one", "visits",
                                   "slots", "no_hits", "images", "field", "mid", "long"])
def test_row_tiles_hold_the_recorded_paths(which):
    """Row tiles whose rows begin and end inside packets and directions: columns
    over the tiles against the recorded paths' (the same products in another FP64
    order: 1e-11, as above), and the reverse mode's sums over the tiles and over the
    segments' slots against the gather over the transposed paths."""
    from paper_1304_4235_amd import Solver
    wl, leaf = _tile_case(which)
    x = torch.tensor(np.random.default_rng(4).uniform(1e-6, 1.0, wl.n))
    s = Solver.from_workload(wl, leaf_size=leaf, record_paths=1)
    s.set_state(x)
    N, hits = s.compute_columns()
    N = N.clone()
    s.set_tuning(tiles=1)
    for _ in range(10):
        s.set_state(x)
        got, h = s.compute_columns()
    assert h == hits and s.timing()["tile_set_total"] > 0
    np.testing.assert_allclose(got.cpu().numpy(), N.cpu().numpy(), rtol=1e-11, atol=0)
    s.set_tuning(tiles=0)
    g = torch.ones(wl.n, dtype=torch.float64, device="cuda")
    dn = []
    for mode in (0, 1, 2):
        s.set_tuning(adjoint_scatter=mode)
        s.forward(2)
        dn.append(s.backward(g, None)[1].cpu().numpy())
    for q in (1, 2):
        np.testing.assert_allclose(dn[q], dn[0], rtol=1e-9, atol=1e-12 * np.abs(dn[0]).max())
    s.close()


def test_row_tiles_need_six_bytes_beside_the_paths():
    """The reverse mode's scatter over row tiles runs where the path buffer holds
    the paths and 7 bytes per intersection: nothing else is laid out beside them
    while the tiles are built."""
    from paper_1304_4235_amd import Solver
    wl = W.isothermal_halo(n=8192, n_bins=8, seed=46)
    s = Solver.from_workload(wl, record_paths=1)
    need = s.count_paths()
    s.close()
    s = Solver.from_workload(wl, record_paths=1, path_budget=need["bytes_paths"] + 7 * need["hits"])
    s.set_tuning(keep_columns=0, adjoint_scatter=2)
    lnG, x = s.forward(2)
    s.backward(torch.ones_like(lnG), None)
    assert s.timing()["tile_set_total"] > 0
    s.close()


def test_paths_over_images_beyond_a_word():
    """Images more than 131071 box lengths away along an axis: recorded (the image
    takes a log word per axis), to the traversal's columns and hit lists."""
    from paper_1304_4235_amd import Solver
    out = []
    for paths in (1, 0):
        s = Solver(l_ray=140000.0, box=1.0, record_paths=paths)
        s.set_particles(np.array([[0.5, 0.5, 0.5], [0.75, 0.5, 0.25]], np.float32),
                        np.array([0.3, 0.35], np.float32), np.array([1e12, 2e12], np.float32),
                        np.array([1e-2, 1e-2], np.float32), np.array([1e4, 1e4], np.float32))
        s.set_rays(np.array([[1.0, 0.0, 0.0], [0.0, -1.0, 0.0], [0.0, 0.0, -1.0]]))
        s.set_spectrum(np.array([6e-18]), np.array([1e5]))
        s.build_tree()
        N, hits = s.compute_columns()
        out.append((N.cpu().numpy(), hits))
        if paths:
            off, j, fac = s.path_rows([0, 1])
            ho, hj, _, hf = s.hits_rows([0, 1])
            np.testing.assert_array_equal(off, ho)
            np.testing.assert_array_equal(j, hj)
            np.testing.assert_array_equal(fac, hf)
        s.close()
    assert out[0][1] == out[1][1] >= 6 * 140000
    np.testing.assert_allclose(out[0][0], out[1][0], rtol=1e-9)


@pytest.mark.parametrize("near_far", [0, 1])
def test_an_overflowing_particle_blocks_its_rays_only(near_far):
    """A density so large that a particle's content leaves the FP32 range (valid
    input): the rays that meet it get an infinite column, as the traversal gives
    them, and no ray becomes NaN."""
    from paper_1304_4235_amd import Solver
    wl = W.isothermal_halo(n=900, n_bins=4, seed=31)
    mu = wl.mu.astype(np.float32).copy()
    nH = wl.n_H.astype(np.float32).copy()
    big = [17, 500, 899]
    mu[big] = 1e38
    dense = nH.copy()
    dense[big] *= 1e6
    out = []
    for paths in (1, 0):
        s = Solver(l_ray=wl.l_ray, box=0.0, record_paths=paths)
        s.set_particles(wl.pos, wl.h, mu, nH, wl.T)
        s.set_rays(wl.dirs)
        s.set_spectrum(wl.sigma, wl.w)
        s.set_scheme(near_far)
        s.build_tree()
        s.set_density(torch.tensor(dense))
        s.set_state(torch.full((wl.n,), 0.5, dtype=torch.float64))
        N, _ = s.compute_columns()
        N = N.cpu().numpy()
        if near_far:
            N = np.concatenate([N, s.near_columns().cpu().numpy()])
        out.append(N)
        s.close()
    assert not np.isnan(out[1]).any() and np.isinf(out[1]).any()
    np.testing.assert_array_equal(np.isinf(out[0]), np.isinf(out[1]))
    np.testing.assert_allclose(out[0], out[1], rtol=1e-11)


@pytest.mark.parametrize("queue", [1, 0])
@pytest.mark.parametrize("which", ["one", "packet_plus_one", "slots", "images", "field", "rays"])
def test_pieces_of_every_size_give_the_same_paths(which, queue):
    """From the least buffer to one that holds the whole log: pieces of single units,
    packets, one direction and several directions, by the walk's queues or by a wave
    to a unit, and recordings of a tree whose sizes are known, are not, or are the
    last tree's: the same columns bit for bit."""
    from paper_1304_4235_amd import Solver
    if which == "rays":                                  # many directions of few packets
        wl, leaf = W.uniform_lattice(n_side_lattice=7, box=20.0, l_ray=30.0, n_side=4), 0
    else:
        wl, leaf = _case(which)
    x = torch.tensor(np.random.default_rng(5).uniform(1e-6, 1.0, wl.n))
    s = Solver.from_workload(wl, leaf_size=leaf, record_paths=1)
    need = s.count_paths()
    s.set_state(x)
    N = s.compute_columns()[0].clone()
    s.close()
    for extra in (0.0, 0.15, 0.6, 2.0, 5.0):
        t = Solver.from_workload(wl, leaf_size=leaf, record_paths=1, build=False,
                                 path_budget=need["bytes_paths"] + int(extra * need["hits"]))
        t.set_tuning(packet_queue=queue)
        for k in range(3):
            t.build_tree()                               # counted, then the last tree's sizes
            if k == 2:
                t.set_tuning(one_pass=0)                 # a walk for the sizes
            t.set_state(x)
            got, h = t.compute_columns()
            assert h == need["hits"] == t.timing()["path_hits"]
            assert torch.equal(got, N), (extra, k)
        t.close()
