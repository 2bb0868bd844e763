"""Calls whose kernels would take a grid of 2^32 threads or more, which HIP
launches cut short, without an error: a small array with very many (time, channel) cells."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
FLUX = {"point_flux": synth._pl(0.05, 50.0), "shapelet_sref": synth._lu(20.0, 200.0), "tau": 20.0}


def test_points_of_a_small_array():
    """24 antennas, 3.4e7 cells: by antenna, four channels a workgroup, 8.4e6
    workgroups of 512 threads."""
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    rng = np.random.default_rng(2)
    obs = synth.make_obs(rng, 24, 32800, synth.channels(182e6, 10e3, 1024), dt_s=0.5)
    sky = synth.make_sky(rng, n_point=96, n_gauss=0, shapelet_nmax=[], cap_rad=math.radians(5.0), **FLUX)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            vis = torch.empty((obs.n_time, obs.n_bl, obs.n_chan), dtype=torch.complex64, device="cuda")
            vp.vp_predict(ctx, h.sky, h.obs, vp.VP_PREC_MIXED, vp.VP_C64, vis.data_ptr(), 0)
            torch.cuda.synchronize()
            t = np.array([0, 1, 16384, 32799])
            got = vis[torch.from_numpy(t).to("cuda")].cpu().numpy()
            del vis
    finally:
        vp.vp_destroy_ctx(ctx)
        torch.cuda.empty_cache()
    import dataclasses
    import oracle
    few = dataclasses.replace(obs, n_time=t.size, uvw_m=np.ascontiguousarray(obs.uvw_m[t]))
    err = oracle.error_metric(got, oracle.predict(few, sky), few, sky)
    print("error / total flux %.2e" % err, flush=True)
    assert err <= 1e-6


def test_gains_of_three_tiles():
    """1.7e7 cells of three tiles: the solve takes them in parts."""
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    rng = np.random.default_rng(3)
    obs = synth.make_obs(rng, 3, 16640, synth.channels(182e6, 10e3, 1024), dt_s=0.5)
    sky = synth.make_sky(rng, n_point=1, n_gauss=0, shapelet_nmax=[], cap_rad=math.radians(1.0), **FLUX)
    a1, a2 = synth.antenna_pairs(3)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            data = torch.empty((obs.n_time, obs.n_bl, obs.n_chan), dtype=torch.complex64, device="cuda")
            vp.vp_predict(ctx, h.sky, h.obs, vp.VP_PREC_MIXED, vp.VP_C64, data.data_ptr(), 0)
            torch.cuda.synchronize()
            top = float(data.abs().max())
            data *= 1.21  # gains of 1.1 on every tile
            torch.cuda.synchronize()
            vp.vp_peel(ctx, h.sky, h.obs, a1, a2, 3, 12, vp.VP_PREC_MIXED, vp.VP_C64, data.data_ptr(), 0, 0)
            torch.cuda.synchronize()
            left = float(data.abs().max())
    finally:
        vp.vp_destroy_ctx(ctx)
        torch.cuda.empty_cache()
    print("residual / largest visibility %.2e" % (left / top), flush=True)
    assert left <= 1e-5 * top
