"""Batched form: uneven-size problems (7-point spherical shells and 11-point
oblate shells) solved together in one launch per phase.  Each result must
equal the same problem solved alone by cps_solve (FP32 V-cycles inside FP64
refinement), bit for bit, and the oracle's exact solution to 1e-9."""
import numpy as np
import pytest

import oracle as O
from oracle import direct
from paper_2305_17875_amd import cps, inputs
from paper_2305_17875_amd.inputs import Shell, MAP_OBLATE
from gpu_util import needs_gpu, log, dev, host, rel, torch

pytestmark = [pytest.mark.gpu, needs_gpu]

GRIDS = [
    Shell(16, 16, 16),
    Shell(32, 32, 64, map=MAP_OBLATE, flattening=0.1),
    Shell(16, 16, 32, radial_stretch=2.0),
    Shell(24, 20, 28, map=MAP_OBLATE, flattening=0.15),
    Shell(32, 32, 32),
    Shell(16, 16, 16, map=MAP_OBLATE, flattening=0.05),
    Shell(32, 32, 64, radial_stretch=2.0),
    # rings of 64 / 128 cells per parity: row-pair kernels; the single solve
    # forms the CG direction inside the product, the batch in its own pass
    Shell(16, 16, 128, radial_stretch=2.0),
    Shell(8, 12, 256),
]


def rhs_of(i, g):
    return inputs.smoothed_noise(g.shape, seed=100 + i)


def alone(g, b, smoother=0):
    s = cps.Solver(g, precision=1, accel=1, smoother=smoother)
    try:
        r = s.solve(dev(b).flatten())
        return host(r.p).reshape(g.shape), r
    finally:
        s.close()


def test_batch_equals_alone_and_oracle():
    log("batch", len(GRIDS))
    rhs = [rhs_of(i, g) for i, g in enumerate(GRIDS)]
    rhs[5] = np.zeros(GRIDS[5].shape)  # a problem that needs no iteration
    B = cps.Batch(GRIDS)
    try:
        st, p, infos = B.solve([dev(b).flatten() for b in rhs])
        xs = [host(t).reshape(g.shape) for t, g in zip(p, GRIDS)]
        # a second solve on the same batch gives the same bits
        st2, p2, _ = B.solve([dev(b).flatten() for b in rhs])
        for t1, t2 in zip(p, p2):
            assert np.array_equal(host(t1), host(t2))
    finally:
        B.close()
    assert st == cps.CPS_OK
    for i, (g, b, x, info) in enumerate(zip(GRIDS, rhs, xs, infos)):
        xa, ra = alone(g, b)
        assert info.iterations == ra.iterations, i
        assert np.array_equal(x, xa), (i, np.abs(x - xa).max())
        if i == 5:
            assert info.iterations == 0 and not x.any()
            continue
        G = O.face_metrics(g)
        want = direct.solve_axisym(G, b)
        assert rel(x, want) <= 1e-9, (i, rel(x, want))


def test_batch_retires_diverged_and_capped_problems():
    log("batch errors")
    grids = [Shell(16, 16, 16), Shell(16, 16, 32), Shell(16, 16, 16, map=MAP_OBLATE, flattening=0.1)]
    rhs = [rhs_of(i, g) for i, g in enumerate(grids)]
    rhs[1][2, 3, 4] = np.nan
    B = cps.Batch(grids)
    try:
        st, p, infos = B.solve([dev(b).flatten() for b in rhs])
    finally:
        B.close()
    assert st == cps.CPS_E_DIVERGED
    assert infos[0].iterations > 0 and infos[0].rel_residual <= 1e-10
    assert infos[2].iterations > 0 and infos[2].rel_residual <= 1e-10
    x0, _ = alone(grids[0], rhs[0])
    assert np.array_equal(host(p[0]).reshape(grids[0].shape), x0)
    B = cps.Batch(grids[:1], max_iters=1)
    try:
        st, p, infos = B.solve([dev(rhs[0]).flatten()])
    finally:
        B.close()
    assert st == cps.CPS_E_NOT_CONVERGED and infos[0].iterations == 1
    with pytest.raises(cps.CpsError):
        cps.Batch([Shell(34, 34, 34)])


def test_batch_with_the_automatic_smoother():
    """smoother = 2: the spheres with power-of-two rings run the plane
    smoother as a group of their own, the oblate shells the plane smoother
    with r-theta cross terms as another, the sphere with a 48-cell ring the
    point smoother; every result equals the same problem solved alone with
    the same opts, bit for bit, and the oracle's exact solution to 1e-9."""
    grids = [Shell(16, 16, 32, radial_stretch=2.0), Shell(32, 32, 64, map=MAP_OBLATE,
                                                          flattening=0.1),
             Shell(32, 32, 64), Shell(16, 16, 48), Shell(8, 12, 256),
             Shell(16, 16, 16, map=MAP_OBLATE, flattening=0.05)]
    rhs = [rhs_of(20 + i, g) for i, g in enumerate(grids)]
    log("batch automatic smoother", len(grids))
    B = cps.Batch(grids, smoother=2)
    try:
        st, p, infos = B.solve([dev(b).flatten() for b in rhs])
        xs = [host(t).reshape(g.shape) for t, g in zip(p, grids)]
    finally:
        B.close()
    assert st == cps.CPS_OK
    for i, (g, b, x, info) in enumerate(zip(grids, rhs, xs, infos)):
        xa, ra = alone(g, b, smoother=2)
        assert info.iterations == ra.iterations, i
        assert np.array_equal(x, xa), (i, np.abs(x - xa).max())
        want = direct.solve_axisym(O.face_metrics(g), b)
        assert rel(x, want) <= 1e-9, (i, rel(x, want))
    log("batch automatic smoother iterations", [i.iterations for i in infos])
    assert infos[0].iterations <= 8 and infos[3].iterations > 3 * infos[0].iterations
    assert infos[1].iterations <= 10 and infos[5].iterations <= 10


def test_batch_plane_smoother_on_long_oblate_rings():
    """smoother = 1 for every problem: oblate shells (r-theta cross terms,
    the batched plane group with cross terms) up to the batched form's
    longest ring (n_phi = 512) beside spheres; every result equals the same
    problem solved alone, bit for bit, and the oracle's exact solution to
    1e-9."""
    grids = [Shell(8, 8, 512, map=MAP_OBLATE, flattening=0.1),
             Shell(16, 16, 64, map=MAP_OBLATE, flattening=0.15, radial_stretch=1.5),
             Shell(8, 8, 512, radial_stretch=1.0)]
    rhs = [rhs_of(60 + i, g) for i, g in enumerate(grids)]
    log("batch plane long rings", len(grids))
    B = cps.Batch(grids, smoother=1)
    try:
        st, p, infos = B.solve([dev(b).flatten() for b in rhs])
        xs = [host(t).reshape(g.shape) for t, g in zip(p, grids)]
    finally:
        B.close()
    assert st == cps.CPS_OK
    for i, (g, b, x, info) in enumerate(zip(grids, rhs, xs, infos)):
        xa, ra = alone(g, b, smoother=1)
        assert info.iterations == ra.iterations, i
        assert np.array_equal(x, xa), (i, np.abs(x - xa).max())
        want = direct.solve_axisym(O.face_metrics(g), b)
        assert rel(x, want) <= 1e-9, (i, rel(x, want))


def test_batch_equals_alone_near_fp64_reach():
    """At a tolerance near what FP64 can reach, the conjugate-gradient
    recurrence and the residual of the iterate part, and both forms check
    (and restart from) the latter in the same way: still the same bits."""
    grids = [GRIDS[0], GRIDS[1], GRIDS[7]]
    rhs = [rhs_of(i, g) for i, g in enumerate(grids)]
    tol = 1e-13
    log("batch near fp64 reach")
    B = cps.Batch(grids, max_iters=60)
    try:
        st, p, infos = B.solve([dev(b).flatten() for b in rhs], tol)
        xs = [host(t).reshape(g.shape) for t, g in zip(p, grids)]
    finally:
        B.close()
    for i, (g, b, x, info) in enumerate(zip(grids, rhs, xs, infos)):
        s = cps.Solver(g, precision=1, accel=1, max_iters=60)
        try:
            r = s.solve(dev(b).flatten(), tol)
            xa = host(r.p).reshape(g.shape)
        finally:
            s.close()
        log(i, "iterations", info.iterations, r.iterations, "rel", info.rel_residual,
            r.rel_residual)
        assert info.iterations == r.iterations and info.rel_residual == r.rel_residual, i
        assert np.array_equal(x, xa), (i, np.abs(x - xa).max())


@pytest.mark.parametrize("n_r", [48, 80, 96, 112])
def test_plane_batch_with_wavefronts_that_hold_no_line(n_r):
    """Lines of 3, 5, 6 and 7 wavefronts in batched blocks of 16, on levels
    of three launches a half-sweep and of one, with and without cross terms: the
    idle wavefronts change nothing, each problem has the bits it gets alone."""
    grids = [Shell(n_r, 16, 64), Shell(n_r, 16, 32, map=MAP_OBLATE, flattening=0.1)]
    rhs = [rhs_of(50 + i, g) for i, g in enumerate(grids)]
    log("plane batch", n_r)
    B = cps.Batch(grids, smoother=1)
    try:
        st, p, infos = B.solve([dev(b).flatten() for b in rhs])
        xs = [host(t).reshape(g.shape) for t, g in zip(p, grids)]
    finally:
        B.close()
    assert st == cps.CPS_OK
    for i, (g, b, x, info) in enumerate(zip(grids, rhs, xs, infos)):
        xa, ra = alone(g, b, smoother=1)
        assert info.iterations == ra.iterations, i
        assert np.array_equal(x, xa), (i, np.abs(x - xa).max())
