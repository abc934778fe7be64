"""L-BFGS with one workgroup per box through every stage (boxes of one part of
at most 16384 entries) against the part launches (the same parts, made longer
than that): the same evaluations and iterations, the same analysis.  Sizes
around the entries that a thread holds (4, 8, 12 and 16 of 1024 threads), a
box smaller than a workgroup, one that is too long for the workgroup, boxes of
several sizes, a pair memory that wraps, and stops at different rounds.

The routes differ in the order of sums over at most 16384 entries (1e-13 of a
sum at the worst), which a few iterations amplify by some hundreds: 1e-9 of
the increment."""
import numpy as np
import pytest


pytestmark = pytest.mark.gpu

SPHERE = dict(index=330, nsteps=8, bands=1, pieces=1, ntime=2, overlap_cells=0, overlap_steps=2,
              obs_frac=0.05, obs_every=2)
CASES = {
    "384": dict(SPHERE, nlat=8, nlon=16),
    "4056": dict(SPHERE, nlat=26, nlon=52),
    "4212": dict(SPHERE, nlat=27, nlon=52),
    "8208": dict(SPHERE, nlat=36, nlon=76),
    "12420": dict(SPHERE, nlat=45, nlon=92),
    "16128": dict(SPHERE, nlat=56, nlon=96),
    "16416": dict(SPHERE, nlat=57, nlon=96),
    "bricks": dict(index=331, nlat=40, nlon=70, brick=(3, 4, 6, 30), ntime=2, nsteps=8,
                   overlap_cells=3, overlap_steps=2, obs_frac=0.05, obs_every=2),
}


@pytest.mark.parametrize("which", list(CASES))
def test_one_part_route(which):
    from conftest import custom_problem
    from paper_2205_06649_amd.context import Context
    p = custom_problem(CASES[which])
    out = []
    for entries in (16384, 1 << 20):
        ctx = Context(p, "fp64")
        ctx.set_solver_parts(entries)
        if which.isdigit():
            assert all(3 * int(i[1]) * int(i[3]) == int(which) for i in ctx.info)
        xa, rep, _, _ = ctx.solve(max_outer=2, max_iter=8, outer_tol=0.0, lbfgs_m=3, grad_rtol=0.05)
        out.append((xa, rep.total_evals, rep.lbfgs_iters, rep.J_final, rep.gnorm_ratio_max))
        ctx.close()
    a, b = out
    err = np.linalg.norm(a[0] - b[0]) / np.linalg.norm(b[0] - p.xb0)
    print(f"{which}: evals {a[1]} iterations {a[2]} difference {err:.1e}", flush=True)
    assert a[1:3] == b[1:3]
    assert err <= 1e-9
    assert abs(a[3] - b[3]) <= 1e-9 * abs(b[3]) and abs(a[4] - b[4]) <= 1e-6 * b[4]
