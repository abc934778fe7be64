"""FP64 sweeps over several levels per launch (execution mode 0) against the
step kernels (mode 1, one launch per box and level): every result bit for
bit, where the blocks can go wrong: whole boxes and boxes cut into blocks (one
to six passes, halos of several rows), boxes spanning the circle with one or
both poles, rows shorter than a wave, boxes of different sizes and ragged last
tiles, one-step intervals, and observations given in any order."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

BASE = dict(index=300, nlat=40, nlon=80, nsteps=16, bands=2, pieces=2, ntime=2, overlap_cells=2,
            overlap_steps=2, obs_frac=0.05, obs_every=3)
CASES = {
    "whole": {},
    "band": dict(bands=3, pieces=1, nlat=33, nlon=64),
    "sphere": dict(bands=1, pieces=1, nlat=24, nlon=48, overlap_cells=0, ntime=2),
    # three passes, in one frame and in two
    "three_two": dict(bands=1, pieces=1, nlat=40, nlon=64, overlap_cells=0, ntime=2),
    "three_one": dict(bands=8, pieces=8, nlat=320, nlon=480, overlap_cells=3, nsteps=22, ntime=2),
    "three_cut": dict(bands=8, pieces=8, nlat=384, nlon=528, overlap_cells=3, nsteps=22, ntime=2),
    "cut": dict(nlat=96, nlon=192, nsteps=30),
    "six_passes": dict(nlat=134, nlon=268, bands=2, pieces=2, overlap_cells=4, nsteps=24, ntime=2),
    "many": dict(nlat=270, nlon=1072, bands=4, pieces=8, overlap_cells=3, nsteps=14, ntime=8,
                 overlap_steps=1),
    "odd": dict(nlat=97, nlon=190, bands=3, pieces=3, nsteps=23, ntime=3, overlap_cells=3),
    "bricks": dict(nlat=160, nlon=320, brick=(4, 6, 24, 96), nsteps=20, overlap_cells=3),
    "narrow": dict(nlat=64, nlon=256, bands=2, pieces=32, nsteps=20),
    "tall": dict(nlat=200, nlon=40, bands=1, pieces=2, nsteps=20, overlap_cells=3),
    "one_step": dict(nsteps=3, ntime=3, overlap_steps=1, obs_every=1),
}


def _problem(which):
    spec = synth.make_spec(dict(BASE, **CASES[which]))
    flat = spec.truth0.reshape(3, -1)
    vals = flat[spec.obs_field.astype(np.int64), spec.obs_cell.astype(np.int64)] + \
        spec.obs_sigma * spec.obs_noise
    order = np.random.default_rng(5).permutation(spec.nobs)
    return spec.replace(obs_value=vals[order], obs_step=spec.obs_step[order],
                        obs_cell=spec.obs_cell[order], obs_field=spec.obs_field[order],
                        obs_sigma=spec.obs_sigma[order], obs_noise=spec.obs_noise[order])


@pytest.mark.parametrize("which", list(CASES))
def test_blocks_equal_step_kernels(which):
    import torch
    from paper_2205_06649_amd.context import Context
    p = _problem(which)
    ctx = Context(p, "fp64")
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

    ctx.set_timing(True)
    blocks = everything()
    launches = ctx.get_timing()
    ctx.set_timing(False)
    # without phase timing both sweeps of whole boxes go in one launch
    J, g = ctx.cost_grad(x)
    blocks.update(J_untimed=J, grad_untimed=g, adjoint_untimed=ctx.adjoint())
    ctx.set_exec_mode(1)
    steps = everything()
    nlev = max(int(i[5]) for i in ctx.info)
    print(f"{which}: {nlev} levels, {launches['fwd_launches']:.0f} forward and "
          f"{launches['adj_launches']:.0f} adjoint launches", flush=True)
    assert launches["fwd_launches"] < nlev - 1 or nlev <= 4     # the blocks ran
    steps.update(J_untimed=steps["J"], grad_untimed=steps["grad"], adjoint_untimed=steps["cost_adjoint"])
    for k in blocks:
        assert torch.equal(blocks[k], steps[k]), k
        assert torch.isfinite(blocks[k]).all(), k
    ctx.close()
