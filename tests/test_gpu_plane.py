"""The zebra (r, phi)-plane smoother on the GPU (Fourier transform along phi
+ Thomas along r) against the oracle's exact block Gauss-Seidel solves
(sparse LU of every (r, phi) plane), its V-cycle against the oracle's plane
V-cycle, and solves against the oracle's exact solution; for the 7-point
operator and for the oblate shell's 11-point one (r-theta cross terms,
whose r-lines are tridiagonal but not symmetric)."""
import numpy as np
import pytest

import oracle as O
from oracle import direct, plane
from paper_2305_17875_amd import cps, inputs
from paper_2305_17875_amd.inputs import Shell, MAP_OBLATE, MAP_IDENTITY, MAP_TRIAXIAL
from gpu_util import needs_gpu, log, dev, host, rel, relmax, torch

pytestmark = [pytest.mark.gpu, needs_gpu]

CASES = [
    ("sphere-stretch-8x8x64", Shell(8, 8, 64, radial_stretch=2.0)),
    ("sphere-6x10x32", Shell(6, 10, 32)),           # 5 rows of each parity
    ("sphere-8x6x128", Shell(8, 6, 128, radial_stretch=2.0)),
    ("sphere-4x4x2048", Shell(4, 4, 2048)),         # the longest ring (1024 per parity)
    ("identity-8x8x32", Shell(8, 8, 32, map=MAP_IDENTITY)),
    ("oblate-8x8x32", Shell(8, 8, 32, map=MAP_OBLATE, flattening=0.1)),
    ("oblate-stretch-6x10x64", Shell(6, 10, 64, map=MAP_OBLATE, flattening=0.15,
                                     radial_stretch=1.5)),
    ("oblate-sphere-full-8x8x16", Shell(8, 8, 16, map=MAP_OBLATE, flattening=0.2,
                                        theta0=0.0, theta1=np.pi)),
    ("oblate-4x6x1024", Shell(4, 6, 1024, map=MAP_OBLATE, flattening=0.1)),
]


@pytest.fixture(scope="module", params=CASES, ids=[c[0] for c in CASES])
def case(request):
    name, g = request.param
    log("plane", name)
    s = cps.Solver(g, precision=0, accel=0, smoother=1)
    mg = O.Multigrid(g)
    yield name, g, s, mg
    s.close()


def test_half_sweeps_match_block_gauss_seidel(case):
    """Per entry to 1e-11 relative: the transform of a ring of up to 2048
    cells adds ~log2(n) roundings, amplified by the plane systems' condition
    (phi coupling ~1e3 x the theta coupling on the longest ring)."""
    name, g, s, mg = case
    rng = np.random.default_rng(11)
    for l, shp in enumerate(s.levels[:-1]):
        G = mg.metrics(l)
        sm = plane.PlaneSmoother(G)
        b = rng.standard_normal(shp)
        x = rng.standard_normal(shp)
        for parity in (0, 1):
            want = sm.half_sweep(b, x, parity)
            xd = dev(x).flatten()
            cps.cps_debug_plane_sweep(s.h, l, parity, dev(b).flatten(), xd)
            got = host(xd).reshape(shp)
            assert relmax(got, want) < 1e-11, (l, parity, relmax(got, want))
            x = want


def test_plane_vcycle_matches_oracle(case):
    name, g, s, mg = case
    pm = plane.PlaneMultigrid(mg, nu=2)
    rng = np.random.default_rng(12)
    b = rng.standard_normal(g.shape)
    b -= b.mean()
    x = rng.standard_normal(g.shape) * 0.1
    want = pm.vcycle(b, x)
    xd = dev(x).flatten()
    cps.cps_debug_vcycle(s.h, dev(b).flatten(), xd)
    got = host(xd).reshape(g.shape)
    assert relmax(got, want) < 1e-11, relmax(got, want)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["sphere", "oblate"])
def test_plane_solve_against_exact_and_fewer_cycles(precision, kind):
    if kind == "sphere":
        g = Shell(32, 32, 64, radial_stretch=2.0)
    else:
        g = Shell(32, 32, 64, map=MAP_OBLATE, flattening=0.1, radial_stretch=2.0)
    b = inputs.smoothed_noise(g.shape, 21)
    want = direct.solve_axisym(O.face_metrics(g), b)
    out = {}
    for sm in (0, 1):
        s = cps.Solver(g, precision=precision, accel=1, smoother=sm, max_iters=400)
        try:
            r = s.solve(dev(b).flatten())
            out[sm] = (host(r.p).reshape(g.shape), r)
        finally:
            s.close()
    x, r = out[1]
    assert r.status == cps.CPS_OK and r.rel_residual <= 1e-10
    assert rel(x, want) <= 1e-9, rel(x, want)
    log("plane cycles", kind, precision, out[0][1].iterations, r.iterations)
    assert r.iterations * 3 <= out[0][1].iterations


def test_plane_smoother_rejects_what_it_cannot_do():
    with pytest.raises(cps.CpsError, match="phi-invariant"):
        cps.Solver(Shell(16, 16, 32, map=MAP_TRIAXIAL, flattening=0.1, skew=0.2), smoother=1)
    with pytest.raises(cps.CpsError, match="power of two"):
        cps.Solver(Shell(16, 16, 48), smoother=1)
    with pytest.raises(cps.CpsError, match="n_phi <= 512"):
        cps.cps_batch_setup([cps.make_grid(Shell(4, 4, 1024))], cps.cps_metrics(0),
                            cps.cps_opts(1, 200, 1, 0, 0, 1, None))


def test_plane_graph_replays_equal_eager():
    g = Shell(16, 16, 64, radial_stretch=2.0)
    side = torch.cuda.Stream()
    sg = cps.Solver(g, precision=1, accel=1, smoother=1, stream=side)
    se = cps.Solver(g, precision=1, accel=1, smoother=1, stream=side, eager=True)
    try:
        for k in range(3):
            b = dev(inputs.smoothed_noise(g.shape, 400 + k)).flatten()
            torch.cuda.synchronize()
            xg = host(sg.solve(b).p)
            xe = host(se.solve(b).p)
            assert np.array_equal(xg, xe), k
    finally:
        sg.close()
        se.close()


def test_service_with_plane_smoother_recomputes_pivots_on_remap():
    """The service with smoother = 1 and one slot: three sphere stretchings
    of one shape share a pooled hierarchy, whose metrics, coarse inverse and
    plane pivots are recomputed in place for each new map; every result
    equals a fresh solve bit for bit, and the footprint estimate covers the
    resident hierarchy."""
    shape = (16, 16, 64)
    gs = [Shell(*shape, radial_stretch=s) for s in (0.0, 2.0, 1.0)]
    reqs = [(g, inputs.smoothed_noise(shape, 60 + i)) for i, g in enumerate(gs)]
    log("plane service remap")
    svc = cps.Service(1 << 30, max_slots=1, precision=1, smoother=1)
    try:
        fp = svc.footprint(gs[0])
        out = [svc.wait(svc.submit(g, b)) for g, b in reqs]
        st = svc.stats()
    finally:
        svc.close()
    for i, ((g, b), (status, p, info)) in enumerate(zip(reqs, out)):
        assert status == cps.CPS_OK, i
        s = cps.Solver(g, precision=1, accel=1, smoother=1)
        try:
            r = s.solve(dev(b).flatten())
            xa = host(r.p).reshape(shape)
        finally:
            s.close()
        assert info.iterations == r.iterations, i
        assert np.array_equal(p, xa), (i, np.abs(p - xa).max())
    assert st["hierarchies_built"] == 1 and st["hierarchies_reused"] == 2, st
    assert st["map_rebuilds"] == 2, st
    assert 0 < st["hbm_in_use"] <= fp, (st["hbm_in_use"], fp)


def test_automatic_smoother_in_the_service():
    """smoother = 2: the hierarchies of a sphere and of an oblate shell (r-theta
    cross terms) take the plane smoother, a triaxial shell's the point
    smoother; each result equals the same problem solved alone with the same
    opts, bit for bit, and the axisymmetric ones need fewer cycles than with
    the point smoother."""
    reqs = [(Shell(16, 16, 32, radial_stretch=2.0), inputs.smoothed_noise((16, 16, 32), 70)),
            (Shell(16, 16, 32, map=MAP_OBLATE, flattening=0.1),
             inputs.smoothed_noise((16, 16, 32), 71)),
            (Shell(32, 32, 64, radial_stretch=2.0), inputs.smoothed_noise((32, 32, 64), 72)),
            (Shell(16, 16, 32, map=MAP_TRIAXIAL, flattening=0.1, skew=0.2),
             inputs.smoothed_noise((16, 16, 32), 73))]
    log("automatic smoother service")
    svc = cps.Service(1 << 30, max_slots=2, precision=1, smoother=2)
    try:
        out = [svc.wait(svc.submit(g, b)) for g, b in reqs]
    finally:
        svc.close()
    for i, ((g, b), (status, p, info)) in enumerate(zip(reqs, out)):
        assert status == cps.CPS_OK, i
        its = {}
        for sm in (2, 0):
            s = cps.Solver(g, precision=1, accel=1, smoother=sm)
            try:
                r = s.solve(dev(b).flatten())
                its[sm] = r.iterations
                if sm == 2:
                    assert np.array_equal(p, host(r.p).reshape(g.shape)), i
                    assert info.iterations == r.iterations, i
            finally:
                s.close()
        log("automatic smoother", g.map, its)
        if g.map == MAP_TRIAXIAL:
            assert its[2] == its[0], its
        else:
            assert 3 * its[2] <= its[0], its


# The elimination's forms by n_r and ring length: one chunk of 16 cells that
# is full, two with a remainder of 2, the most chunks a block holds (16), and
# the streaming form past it; rings whose lines fill a wavefront with one
# theta row (n_phi / 2 >= 32) and shorter ones, and a last wavefront that is
# not full (3 rows of 8 modes).
ELIM = [(16, 6, 16), (18, 6, 64), (34, 4, 16), (128, 4, 64), (256, 4, 32), (256, 6, 4), (258, 4, 16)]


@pytest.mark.parametrize("map_", [MAP_IDENTITY, MAP_OBLATE], ids=["box", "oblate"])
@pytest.mark.parametrize("shape", ELIM, ids=lambda s: "x".join(map(str, s)))
def test_elimination_chunks_and_remainders(shape, map_):
    """One half-sweep of each parity against the oracle's sparse LU, per entry
    to 1e-11 relative.  The shell's gap grows with n_r (a quarter of a length
    unit a cell), so that a plane's system stays well conditioned (theta
    couplings within 1e4 of the radial ones): n_r eps cond ~ 256 * 2e-16 * 1e2."""
    f = 0.1 if map_ == MAP_OBLATE else 0.0
    g = Shell(*shape, map=map_, flattening=f, r_inner=1.5, r_outer=1.5 + 0.25 * shape[0])
    s = cps.Solver(g, precision=0, accel=0, smoother=1, n_levels=2)
    try:
        G = O.face_metrics(g)
        sm = plane.PlaneSmoother(G)
        rng = np.random.default_rng(5)
        b = rng.standard_normal(shape)
        x = rng.standard_normal(shape)
        for parity in (0, 1):
            want = sm.half_sweep(b, x, parity)
            xd = dev(x).flatten()
            cps.cps_debug_plane_sweep(s.h, 0, parity, dev(b).flatten(), xd)
            got = host(xd).reshape(shape)
            log("elimination", map_, shape, parity, relmax(got, want))
            assert relmax(got, want) < 1e-11, (parity, relmax(got, want))
            x = want
    finally:
        s.close()


# A half-sweep in one launch: (r, phi) planes of up to 1024 complex values on
# rings of up to 256, here at that size by n_r and by ring and one step above
# it (three launches, rings within and past a wavefront's lines), the shortest
# ring, and a last group of rings that is not full.
ROWS = [(32, 4, 64), (34, 4, 64), (64, 6, 32), (66, 4, 32), (4, 6, 512), (6, 4, 512), (256, 4, 4),
        (18, 6, 16)]


@pytest.mark.parametrize("map_", [MAP_IDENTITY, MAP_OBLATE], ids=["box", "oblate"])
@pytest.mark.parametrize("shape", ROWS, ids=lambda s: "x".join(map(str, s)))
def test_half_sweep_launch_forms(shape, map_):
    """Bounds and geometry as test_elimination_chunks_and_remainders."""
    test_elimination_chunks_and_remainders(shape, map_)


@pytest.mark.parametrize("shape", [(64, 8, 64), (128, 8, 128)], ids=["one-launch", "three-launch"])
@pytest.mark.parametrize("map_", [MAP_IDENTITY, MAP_OBLATE], ids=["box", "oblate"])
def test_vcycle_starts_coarse_levels_from_zero(shape, map_):
    """The first half-sweep of a coarse level takes its iterate as zero and
    does not read it, in either launch form: the second of two V-cycles, whose
    coarse arrays hold the first's values, against the oracle's to 1e-11
    relative (three levels of the half-sweeps' 1e-12)."""
    f = 0.1 if map_ == MAP_OBLATE else 0.0
    g = Shell(*shape, map=map_, flattening=f, r_inner=1.5, r_outer=1.5 + 0.25 * shape[0])
    s = cps.Solver(g, precision=0, accel=0, smoother=1, n_levels=3)
    try:
        mg = O.Multigrid(g, n_levels=3)
        pm = plane.PlaneMultigrid(mg, nu=2)
        rng = np.random.default_rng(6)
        x = rng.standard_normal(shape) * 0.1
        for _ in range(2):
            b = rng.standard_normal(shape)
            b -= b.mean()
            want = pm.vcycle(b, x)
            xd = dev(x).flatten()
            cps.cps_debug_vcycle(s.h, dev(b).flatten(), xd)
            x = host(xd).reshape(shape)
            log("zero start", map_, shape, relmax(x, want))
            assert relmax(x, want) < 1e-11, relmax(x, want)
    finally:
        s.close()


@pytest.mark.parametrize("shape", [(8, 16, 512), (8, 12, 256), (6, 10, 64)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("map_", [MAP_IDENTITY, MAP_OBLATE], ids=["box", "oblate"])
def test_transfers_of_the_even_rows(shape, map_):
    """After pre-smoothing the odd rows' equations hold, and post-smoothing
    overwrites those rows first: residual, restriction and correction take the
    even ones only.  The forms by ring and rows (row pairs with the row-wise and
    the general restriction, neither), a V-cycle against the oracle's, which
    takes all rows: to 1e-11 relative."""
    g = Shell(*shape, map=map_, flattening=0.1 if map_ == MAP_OBLATE else 0.0)
    s = cps.Solver(g, precision=0, accel=0, smoother=1, n_levels=2 if shape[2] == 64 else 3)
    try:
        mg = O.Multigrid(g, n_levels=2 if shape[2] == 64 else 3)
        rng = np.random.default_rng(7)
        b = rng.standard_normal(shape)
        b -= b.mean()
        x = rng.standard_normal(shape) * 0.1
        want = plane.PlaneMultigrid(mg, nu=2).vcycle(b, x)
        xd = dev(x).flatten()
        cps.cps_debug_vcycle(s.h, dev(b).flatten(), xd)
        err = relmax(host(xd).reshape(shape), want)
        log("even rows", map_, shape, err)
        assert err < 1e-11, err
    finally:
        s.close()
