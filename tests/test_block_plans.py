"""Plans of the FP64 block sweeps (host)."""
import time

import numpy as np
import pytest

import synth

BASE = dict(index=350, overlap_cells=3, overlap_steps=2, obs_frac=0.02, obs_every=3)


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
