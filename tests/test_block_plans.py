"""The FP64 block sweeps by the plan that they run: whole boxes and boxes cut
into blocks, blocks of one to six passes of 1024 cells, one and two level frames
on chip, boxes spanning the circle alone and beside cut ones, and plans of which
only some sweeps run in blocks (the others in step kernels).  The plan of every
case is pinned on the host (256 compute units) and, on the device, every sweep
of it equals the step kernels (mode 1, one launch per box and level) bit for bit.
Solves, whose evaluations and products leave out the boxes that have stopped,
are compared the same way."""
import time

import numpy as np
import pytest

import synth

BASE = dict(index=350, overlap_cells=3, overlap_steps=2, obs_frac=0.02, obs_every=3)
# levels per launch, passes, frames, blocks, sweeps in blocks (1 forward, 2 cost adjoint, 4
# forced adjoint, 8 Gauss-Newton product, 16 tangent linear)
CASES = {
    "whole_1_two": (dict(nlat=30, nlon=26, nsteps=5, bands=3, pieces=2, ntime=1), (6, 1, 2, 6, 31)),
    "whole_2_two": (dict(nlat=27, nlon=210, nsteps=4, bands=1, pieces=6, ntime=1), (5, 2, 2, 6, 31)),
    "whole_3_two": (dict(nlat=132, nlon=504, nsteps=20, bands=6, pieces=6, ntime=4), (10, 3, 2, 144, 31)),
    "whole_3_one": (dict(nlat=726, nlon=108, nsteps=20, bands=6, pieces=6, ntime=4), (10, 3, 1, 144, 31)),
    "whole_4_one": (dict(nlat=445, nlon=192, nsteps=20, bands=5, pieces=8, ntime=4, overlap_cells=4,
                         overlap_steps=3), (12, 4, 1, 160, 31)),
    "whole_5_one": (dict(nlat=465, nlon=272, nsteps=20, bands=5, pieces=8, ntime=4, overlap_cells=4),
                    (10, 5, 1, 160, 31)),
    "whole_6_one": (dict(nlat=348, nlon=444, nsteps=16, bands=6, pieces=6, ntime=4, overlap_cells=4,
                         overlap_steps=1), (7, 6, 1, 144, 31)),
    "cut_1_two": (dict(nlat=24, nlon=60, nsteps=10, bands=1, pieces=2, ntime=2, overlap_cells=4,
                       overlap_steps=1), (3, 1, 2, 16, 31)),
    "cut_2_two": (dict(nlat=20, nlon=156, nsteps=24, bands=1, pieces=2, ntime=1), (6, 2, 2, 14, 31)),
    "cut_2_one": (dict(nlat=27, nlon=526, nsteps=8, bands=2, pieces=2, ntime=2, overlap_steps=3),
                  (4, 2, 1, 140, 31)),
    "cut_2_some": (dict(nlat=28, nlon=590, nsteps=4, bands=1, pieces=2, ntime=1, overlap_cells=4),
                   (3, 2, 1, 68, 1)),
    "cut_2_fwd_tlm": (dict(nlat=28, nlon=852, nsteps=5, bands=2, pieces=3, ntime=1, overlap_cells=2,
                           overlap_steps=1), (3, 2, 1, 108, 17)),
    "cut_3_two": (dict(nlat=180, nlon=484, nsteps=10, bands=6, pieces=4, ntime=2, overlap_cells=4,
                       overlap_steps=3), (4, 3, 2, 192, 31)),
    "cut_3_one": (dict(nlat=13, nlon=2070, nsteps=12, bands=1, pieces=9, ntime=2, overlap_cells=4,
                       overlap_steps=4), (5, 3, 1, 216, 31)),
    "cut_4_one": (dict(nlat=37, nlon=1028, nsteps=20, bands=2, pieces=4, ntime=4), (5, 4, 1, 192, 31)),
    "cut_4_some": (dict(nlat=37, nlon=1740, nsteps=16, bands=1, pieces=6, ntime=2, overlap_cells=2,
                        overlap_steps=1), (5, 4, 1, 192, 5)),
    "cut_5_one": (dict(nlat=66, nlon=1110, nsteps=16, bands=6, pieces=3, ntime=4), (4, 5, 1, 144, 31)),
    "cut_6_one": (dict(nlat=228, nlon=756, nsteps=16, bands=4, pieces=6, ntime=4, overlap_steps=3),
                  (8, 6, 1, 192, 31)),
    "span_1_two": (dict(nlat=20, nlon=36, nsteps=4, bands=2, pieces=1, ntime=1), (5, 1, 2, 2, 31)),
    "span_2_two": (dict(nlat=43, nlon=30, nsteps=4, bands=1, pieces=1, ntime=1, overlap_cells=0),
                   (5, 2, 2, 1, 31)),
    "span_2_some": (dict(nlat=27, nlon=92, nsteps=112, bands=2, pieces=1, ntime=8, overlap_cells=4),
                    (19, 2, 2, 16, 15)),
    "span_3_two": (dict(nlat=273, nlon=44, nsteps=48, bands=7, pieces=1, ntime=8, overlap_cells=4),
                   (11, 3, 2, 56, 31)),
    "span_3_some": (dict(nlat=33, nlon=182, nsteps=48, bands=3, pieces=1, ntime=2, overlap_cells=2,
                         overlap_steps=1), (26, 3, 1, 6, 1)),
    "span_3_one": (dict(nlat=192, nlon=150, nsteps=64, bands=16, pieces=1, ntime=8), (13, 3, 1, 128, 31)),
    "span_4_one": (dict(nlat=400, nlon=100, nsteps=64, bands=16, pieces=1, ntime=8), (13, 4, 1, 128, 31)),
    "span_5_one": (dict(nlat=512, nlon=128, nsteps=96, bands=16, pieces=1, ntime=16, obs_frac=0.005),
                   (11, 5, 1, 256, 31)),
    "span_6_one": (dict(nlat=320, nlon=200, nsteps=64, bands=16, pieces=1, ntime=8), (13, 6, 1, 128, 31)),
    # polar caps of one piece beside bands of three: caps whole, the others cut
    "caps_cut": (dict(nlat=120, nlon=160, nsteps=24, bands=4, pieces=3, ntime=2, caps=True),
                 (12, 2, 2, 116, 31)),
}


def _problem(cfg, south_only=False):
    cfg = dict(BASE, **cfg)
    caps = cfg.pop("caps", False)
    spec = synth.make_spec(cfg)
    if caps:
        edges = np.array(spec.band_lat_edges)
        edges[1], edges[-2] = 6, cfg["nlat"] - 6
        inner = spec.piece_lon_edges[:cfg["pieces"] + 1]
        spec = spec.replace(
            band_lat_edges=edges, band_npieces=np.array([1] + [cfg["pieces"]] * (cfg["bands"] - 2) + [1],
                                                        spec.band_npieces.dtype),
            piece_lon_edges=np.concatenate([[0, cfg["nlon"]]] + [inner] * (cfg["bands"] - 2) +
                                           [[0, cfg["nlon"]]]).astype(spec.piece_lon_edges.dtype))
    flat = spec.truth0.reshape(3, -1)
    vals = flat[spec.obs_field.astype(np.int64), spec.obs_cell.astype(np.int64)] + \
        spec.obs_sigma * spec.obs_noise
    order = np.random.default_rng(5).permutation(spec.nobs)
    if south_only:
        order = order[spec.obs_cell[order] < cfg["nlat"] * cfg["nlon"] // 2]
    return spec.replace(obs_value=vals[order], **{k: getattr(spec, k)[order] for k in (
        "obs_step", "obs_cell", "obs_field", "obs_sigma", "obs_noise")})


def _pinned(which, plan):
    assert tuple(plan[k] for k in ("levels", "passes", "frames", "blocks", "sweeps")) == CASES[which][1], plan


@pytest.mark.parametrize("which", list(CASES))
def test_plan(which):
    from paper_2205_06649_amd.descriptors import Plan
    p = Plan(_problem(CASES[which][0]))
    _pinned(which, p.block_sweeps(256))
    p.close()


@pytest.mark.parametrize("pieces", [2, 4])
def test_plan_of_wide_boxes_is_quick(pieces):
    """No block of a box of 1024 x 1032 cells fits a workgroup, nor one of
    1024 x 520 (a one-tile block with its halo rows exceeds the LDS): known at
    once, where trying every cut took 20 and 4 seconds."""
    from paper_2205_06649_amd.descriptors import Plan
    p = Plan(_problem(dict(nlat=1024, nlon=2048, nsteps=50, bands=1, pieces=pieces, ntime=1,
                           overlap_cells=4, overlap_steps=0, obs_frac=1e-5, obs_every=25)))
    t = time.perf_counter()
    plan = p.block_sweeps(256)
    t = time.perf_counter() - t
    print(pieces, f"{t:.4f} s", flush=True)
    p.close()
    assert plan["levels"] == 0 and t < 0.5


def _context(p):
    import torch
    from paper_2205_06649_amd.context import Context
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the pinned plans are for 256 compute units")
    return Context(p, "fp64")


@pytest.mark.gpu
@pytest.mark.parametrize("which", list(CASES))
def test_sweeps_equal_step_kernels(which):
    import torch
    ctx = _context(_problem(CASES[which][0]))
    plan = ctx.block_sweeps()
    _pinned(which, plan)
    nlev = max(int(i[5]) for i in ctx.info)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)

    def noise(n):
        return torch.randn(n, generator=gen, device="cuda:0", dtype=torch.float64)

    x = ctx.background_controls() + noise(ctx.ctrl_len)
    dx, force = noise(ctx.ctrl_len), noise(ctx.traj_len)

    def everything():
        J, g = ctx.cost_grad(x)
        return dict(J=J, grad=g, cost_adjoint=ctx.adjoint(), traj=ctx.forward(x),
                    adjoint=ctx.adjoint(force), tangent=ctx.tangent_linear(dx),
                    product=ctx.gn_hessvec(dx))

    print(which, plan, flush=True)
    blocks = everything()
    ctx.set_timing(True)                     # forward and adjoint in launches of their own
    J, g = ctx.cost_grad(x)
    launches = ctx.get_timing()
    ctx.set_timing(False)
    blocks.update(J_timed=J, grad_timed=g)
    # (the step kernels take a launch per level)
    assert launches["fwd_launches"] == (max(1, -(-(nlev - 1) // plan["levels"])) if plan["sweeps"] & 1 else nlev)
    assert launches["adj_launches"] == (-(-nlev // plan["levels"]) if plan["sweeps"] & 2 else nlev)
    ctx.set_exec_mode(1)
    assert ctx.block_sweeps()["levels"] == 0
    steps = everything()
    steps.update(J_timed=steps["J"], grad_timed=steps["grad"])
    for k in blocks:
        assert torch.equal(blocks[k], steps[k]), k
        assert torch.isfinite(blocks[k]).all(), k
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("solver", ["lbfgs", "gn"])
@pytest.mark.parametrize("which", ["whole_2_two", "whole_3_one", "cut_1_two", "cut_4_one",
                                   "cut_2_some", "span_1_two"])
def test_solves_equal_step_kernels(which, solver):
    """Boxes stop at different rounds (no observations in the north) and are
    left out from then on."""
    import torch
    p = _problem(CASES[which][0], south_only=True)
    out = []
    for mode in (0, 1):
        ctx = _context(p)
        if mode == 0:
            _pinned(which, ctx.block_sweeps())
        ctx.set_exec_mode(mode)
        xa, rep, _, xo = ctx.solve(max_outer=2, max_iter=6, outer_tol=0.0, grad_rtol=0.05, cg_max_iter=8,
                                   local_solver=solver, want_controls=True)
        out.append((xa, xo, rep.total_evals, rep.lbfgs_iters, rep.J_final, rep.gnorm_ratio_max))
        ctx.close()
    a, b = out
    print(which, solver, a[2:], flush=True)
    assert a[2:] == b[2:] and np.isfinite(a[0]).all()
    assert np.array_equal(a[0], b[0]) and torch.equal(a[1], b[1])
