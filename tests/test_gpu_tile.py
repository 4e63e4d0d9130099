"""The tile path of small levels (csrc/tile.hpp: 8 x 8 x 8 tiles, the V-cycle's
work on a level in two launches) against the oracle's multigrid, where rings
and walls cut its tiles, and the batched form's bits against the single
solve's."""
import numpy as np
import pytest

import oracle as O
from paper_2305_17875_amd import cps, inputs
from paper_2305_17875_amd.inputs import Shell, MAP_OBLATE, MAP_TRIAXIAL
from gpu_util import needs_gpu, log, dev, host, rel, torch

pytestmark = [pytest.mark.gpu, needs_gpu]

SHAPES = [
    (20, 24, 36),   # the last tile of a ring and of the radial direction half full
    (8, 8, 12),     # a ring shorter than a tile's box, which wraps onto it
    (4, 4, 8),      # one tile, half full in two directions
    (6, 10, 68),    # tiles cut at 6 of 8 planes and 2 of 8 rows; ring remainder 4
    (16, 16, 2048), # a long ring, the most cells of FP32's limit
    (80, 96, 144),  # levels of 138240 (beyond 2^16: rows of part wavefronts) and 17280 cells
]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_one_iteration_matches_oracle(shape, precision):
    """One iteration of conjugate gradients from zero, x = alpha V(b), with at
    least two levels: FP64 to 1e-11 (a V-cycle's sums in another order); FP32
    cycles to 2e-5 (about 20 passes and transfers a level of ~10 roundings of
    6e-8)."""
    n_levels = 2 if shape[0] * shape[1] * shape[2] < 1 << 15 else 0
    g = Shell(*shape, radial_stretch=1.0)
    b = inputs.smoothed_noise(shape, 33)
    s = cps.Solver(g, precision=precision, max_iters=1, n_levels=n_levels,
                   stream=torch.cuda.Stream())
    try:
        x = host(s.solve(dev(b).flatten()).p).reshape(shape)
    finally:
        s.close()
    want = O.Multigrid(g, n_levels=n_levels).solve(b, tol=1e-300, max_iters=1, accel=1)[0]
    err = rel(x, want)
    log("tile", shape, precision, err)
    assert err < (1e-11 if precision == 0 else 2e-5)


def test_batch_equals_alone():
    grids = [Shell(*s, radial_stretch=1.0) for s in SHAPES[:4]]
    rhs = [dev(inputs.smoothed_noise(g.shape, 50 + i)).flatten() for i, g in enumerate(grids)]
    B = cps.Batch(grids, smoother=0)
    try:
        st, p, infos = B.solve(rhs)
    finally:
        B.close()
    assert st == cps.CPS_OK
    for g, b, x, info in zip(grids, rhs, p, infos):
        s = cps.Solver(g, precision=1, smoother=0)
        try:
            r = s.solve(b)
        finally:
            s.close()
        log("tile batch", g.shape, info.iterations, r.iterations)
        assert info.iterations == r.iterations
        assert np.array_equal(host(x), host(r.p)), g.shape


SWEEPS = [(20, 24, 36), (8, 8, 12), (4, 4, 8), (6, 10, 68), (32, 32, 128), (32, 32, 136)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("map_", [MAP_OBLATE, MAP_TRIAXIAL], ids=["oblate", "triaxial"])
@pytest.mark.parametrize("shape", SWEEPS, ids=lambda s: "x".join(map(str, s)))
def test_four_colour_sweeps_match_oracle(shape, map_, precision):
    """Operators with cross terms, point smoother: a launch a sweep up to 2^17
    cells (32 x 32 x 128), tiles cut by rings and walls; above it a launch a
    colour.  Bounds as test_one_iteration_matches_oracle with twice the passes:
    2e-11 and 4e-5."""
    n_levels = 2 if shape[0] * shape[1] * shape[2] < 1 << 15 else 0
    g = Shell(*shape, map=map_, flattening=0.1, skew=0.2 if map_ == MAP_TRIAXIAL else 0.0)
    b = inputs.smoothed_noise(shape, 35)
    s = cps.Solver(g, precision=precision, max_iters=1, n_levels=n_levels,
                   stream=torch.cuda.Stream())
    try:
        x = host(s.solve(dev(b).flatten()).p).reshape(shape)
    finally:
        s.close()
    want = O.Multigrid(g, n_levels=n_levels).solve(b, tol=1e-300, max_iters=1, accel=1)[0]
    err = rel(x, want)
    log("sweep", shape, map_, precision, err)
    assert err < (2e-11 if precision == 0 else 4e-5)


# The outer iteration's launches off the row-pair levels: direction and product
# in one, sums added up by the blocks that use them (the tile path's and the
# marching path's r . z), or by launches (a single level and the plane smoother
# leave no partial sums); rings of whole wavefronts and others.
OUTER = [((32, 32, 32), 0, 0), ((20, 24, 36), 0, 0), ((80, 96, 144), 0, 0), ((4, 7, 128), 0, 1),
         ((16, 16, 32), 1, 0)]


@pytest.mark.parametrize("shape,smoother,n_levels", OUTER,
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_outer_iterations_match_oracle(shape, smoother, n_levels):
    """Four iterations of FP64 conjugate gradients, point smoother: to 1e-10 of
    the oracle's (each iteration's 1e-11 carried on by the later ones); plane
    smoother and single level: a solve to 1e-10, whose residual the oracle forms
    of the answer."""
    g = Shell(*shape, radial_stretch=1.0)
    b = inputs.smoothed_noise(shape, 36)
    few = smoother == 0 and n_levels == 0
    s = cps.Solver(g, precision=0, smoother=smoother, n_levels=n_levels,
                   max_iters=4 if few else 200, stream=torch.cuda.Stream())
    try:
        r = s.solve(dev(b).flatten())
        x = host(r.p).reshape(shape)
    finally:
        s.close()
    if few:
        want = O.Multigrid(g).solve(b, tol=1e-300, max_iters=4, accel=1)[0]
        log("outer", shape, rel(x, want))
        assert rel(x, want) < 1e-10
    else:
        d = b - b.mean()
        res = np.linalg.norm(O.residual(O.face_metrics(g), d, x)) / np.linalg.norm(d)
        log("outer", shape, r.iterations, res)
        assert r.status == cps.CPS_OK and res <= 1.001e-10


@pytest.mark.parametrize("shape,map_,precision", [((16, 16, 24), 1, 0), ((16, 16, 24), 1, 1),
                                                  ((16, 16, 32), MAP_TRIAXIAL, 1)],
                         ids=["fp64", "mixed", "triaxial"])
def test_iterations_launched_ahead_leave_no_trace(shape, map_, precision):
    """A small solve launches an iteration before it has read the last one's
    norm; the eager form does not.  Iterate, count and residual are the same
    bits, wherever the solve ends (a norm, the limit, never) and whatever the
    solve before it on the same handle did."""
    g = Shell(*shape, map=map_, flattening=0.1 if map_ == MAP_TRIAXIAL else 0.0,
              skew=0.2 if map_ == MAP_TRIAXIAL else 0.0)
    side = torch.cuda.Stream()
    for most in (1, 2, 3, 60):
        sa, se = (cps.Solver(g, precision=precision, max_iters=most, stream=side, eager=e)
                  for e in (False, True))
        try:
            for k, tol in enumerate((1e-2, 1e-10, 1e-15, 1e-160, 1e-6)):
                b = dev(inputs.smoothed_noise(shape, 60 + k)).flatten()
                torch.cuda.synchronize()
                ra = sa.solve(b, tol=tol)
                xa = host(ra.p)
                re = se.solve(b, tol=tol)
                log("ahead", shape, most, tol, ra.iterations, ra.status)
                assert (ra.status, ra.iterations, ra.rel_residual) == \
                    (re.status, re.iterations, re.rel_residual)
                assert np.array_equal(xa, host(re.p)), (most, tol)
        finally:
            sa.close()
            se.close()
