"""The marching path of large levels (csrc/march.hpp: more than 2^20 cells, the
V-cycle's work on a level in two launches) against the oracle's multigrid,
where its blocks, segments and chunks end unevenly, and the batched form's
bits against the single solve's."""
import numpy as np
import pytest

import oracle as O
from paper_2305_17875_amd import cps, inputs
from paper_2305_17875_amd.inputs import Shell, MAP_IDENTITY
from gpu_util import needs_gpu, log, dev, host, rel, torch

pytestmark = [pytest.mark.gpu, needs_gpu]

SHAPES = [
    (192, 64, 128),  # a ring of one whole wavefront, which wraps
    (80, 96, 144),   # two segments of 40 and 32 phi pairs; chunks with a remainder
    (128, 88, 112),  # one segment that wraps onto its own halo; half a strip at the wall
    (32, 72, 512),   # five segments; a strip of 8 rows
    (16, 136, 512),  # few planes: one chunk of them all, the halo longer than a wall's distance
    (64, 40, 464),   # segments of the most pairs a wavefront owns (58)
]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_one_iteration_matches_oracle(shape, precision):
    """One iteration of conjugate gradients from zero, x = alpha V(b), on the
    sphere: FP64 to 1e-11 (a V-cycle's sums in another order); FP32 cycles to
    2e-5 (about 20 passes and transfers a level of ~10 roundings of 6e-8)."""
    g = Shell(*shape, radial_stretch=2.0)
    b = inputs.smoothed_noise(shape, 31)
    s = cps.Solver(g, precision=precision, max_iters=1, stream=torch.cuda.Stream())
    try:
        x = host(s.solve(dev(b).flatten()).p).reshape(shape)
    finally:
        s.close()
    want = O.Multigrid(g).solve(b, tol=1e-300, max_iters=1, accel=1)[0]
    err = rel(x, want)
    log("march", shape, precision, err)
    assert err < (1e-11 if precision == 0 else 2e-5)


@pytest.mark.parametrize("precision", [0, 1])
def test_constants_and_walls(precision):
    """The uniform box (r low walls at plane 0, theta walls of both strips): a
    solve to 1e-10 ends with the residual the oracle forms of its answer."""
    g = Shell(32, 72, 512, map=MAP_IDENTITY)
    b = inputs.smoothed_noise(g.shape, 32)
    s = cps.Solver(g, precision=precision, stream=torch.cuda.Stream())
    try:
        r = s.solve(dev(b).flatten())
        x = host(r.p).reshape(g.shape)
    finally:
        s.close()
    assert r.status == cps.CPS_OK
    res = np.linalg.norm(O.residual(O.face_metrics(g), b, x)) / np.linalg.norm(b)
    assert res <= 1.001e-10 and abs(res - r.rel_residual) <= 1e-3 * res, (res, r.rel_residual)


def test_batch_equals_alone():
    """Problems with and without marching levels, point smoother: the batch
    gives each problem the bits it gets alone."""
    grids = [Shell(80, 96, 144, radial_stretch=2.0), Shell(16, 16, 32), Shell(128, 128, 128)]
    rhs = [dev(inputs.smoothed_noise(g.shape, 40 + i)).flatten() for i, g in enumerate(grids)]
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
            assert info.iterations == r.iterations
            assert np.array_equal(host(x), host(r.p)), g.shape
        finally:
            s.close()


@pytest.mark.parametrize("shape", [(80, 96, 144), (64, 40, 464)],
                         ids=lambda s: "x".join(map(str, s)))
def test_intermediate_iterate_needs_no_black_cells(shape):
    """The way down writes only the red cells of its iterate, so a solve must
    not depend on what the black ones hold.  A V-cycle of NaN from a nonzero
    iterate stores its whole residual (rings that are no row pairs) in the
    buffer that later holds that iterate; the same solve before and after it
    gives the same bits."""
    g = Shell(*shape, radial_stretch=2.0)
    b = dev(inputs.smoothed_noise(shape, 33)).flatten()
    s = cps.Solver(g, max_iters=3, stream=torch.cuda.Stream())
    try:
        before = s.solve(b)
        x = host(before.p)
        nan = torch.full((g.cells,), float("nan"), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        cps.cps_debug_vcycle(s.h, nan, nan.clone())
        after = s.solve(b)
        log("march black cells", shape, before.rel_residual, after.rel_residual)
        assert after.status == before.status == cps.CPS_E_NOT_CONVERGED
        assert np.array_equal(host(after.p), x)
    finally:
        s.close()


def test_batch_with_a_finest_level_too_large_to_march():
    """2^28 cells run pass by pass above a level that marches: the batch takes
    the correction from where that level left it, so two iterations give the
    bits of the problem alone."""
    g = Shell(1024, 512, 512, radial_stretch=2.0)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(34)
    b = torch.randn(g.cells, generator=gen, dtype=torch.float64, device="cuda")
    log("march batch", g.shape)
    B = cps.Batch([g], smoother=0, max_iters=2)
    try:
        st, p, infos = B.solve([b])
        x = p[0].clone()
    finally:
        B.close()
    s = cps.Solver(g, precision=1, smoother=0, max_iters=2)
    try:
        r = s.solve(b)
        log("march batch", infos[0].rel_residual, r.rel_residual)
        assert st == r.status == cps.CPS_E_NOT_CONVERGED
        assert infos[0].rel_residual == r.rel_residual and torch.equal(x, r.p)
    finally:
        s.close()
        torch.cuda.empty_cache()


@pytest.mark.parametrize("precision", [0, 1])
def test_a_field_near_the_byte_limit(precision):
    """512 x 960 x 512 cells, 1.9 GiB an FP64 field of the 2 GiB that the
    marching path addresses: the solve converges, and the residual of its
    answer, which other kernels form, meets the tolerance."""
    g = Shell(512, 960, 512, radial_stretch=2.0)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(35)
    b = torch.randn(g.cells, generator=gen, dtype=torch.float64, device="cuda")
    b -= b.mean()
    s = cps.Solver(g, precision=precision, max_iters=200)
    try:
        r = s.solve(b, tol=1e-8)
        log("march byte limit", precision, r.status, r.iterations, r.rel_residual)
        assert r.status == cps.CPS_OK and r.rel_residual <= 1e-8
        p = r.p.view(g.shape)
        assert bool(torch.isfinite(p).all()) and abs(float(p.mean())) <= 1e-12 * float(p.abs().max())
    finally:
        s.close()
        torch.cuda.empty_cache()
