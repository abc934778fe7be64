"""Device memory of a context per observation: the code, value and weight of an
entry (20 B) in every box that holds it, and nothing per (tile, level) bin
where no kernel reads it.  The masks of the block sweeps (112 B per bin with
entries) belong to FP64 contexts that run them; here FP32, and FP64 with boxes
too wide for a block."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CFG = dict(index=340, nlat=512, nlon=1024, nsteps=95, bands=2, pieces=2, ntime=1, overlap_cells=2,
           overlap_steps=0, obs_frac=0.004, obs_every=1)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_observation_memory(precision):
    import torch
    from paper_2205_06649_amd.context import Context
    spec = synth.make_spec(CFG)
    h = np.flatnonzero(spec.obs_field == 0)

    def used(keep):
        p = spec.replace(obs_value=spec.truth0.reshape(3, -1)[0, spec.obs_cell[keep]],
                         **{k: getattr(spec, k)[keep] for k in ("obs_step", "obs_cell", "obs_field",
                                                                "obs_sigma", "obs_noise")})
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        ctx = Context(p, precision)
        after = torch.cuda.mem_get_info()[0]
        ctx.close()
        return before - after

    used(h[:1])                              # (the library's own first-time memory)
    few, many = used(h[:1]), used(h)
    # 1.03: entries in two boxes' overlap; three arrays, each rounded up to at most 2 MiB
    bound = 20 * 1.03 * len(h) + 3 * (2 << 20)
    print(precision, len(h), "observations:", many - few, "bytes, bound", bound, flush=True)
    assert many - few <= bound
