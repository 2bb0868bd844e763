"""Shapelets at sizes that the dispatch gives to the node kernels (k_shp_nodes,
k_shp_nodes64; tests/test_shapelet_nodes.py holds sizes that go to the channel
kernels).  Up to four points beside shapelets go along with the node kernels'
outputs, without a launch of their own: that the points' launch count is 0 shows
which kernel ran.  Bars: the paths' own, 1e-6 and 1e-11 of the total flux (1e-6
for complex64)."""
import dataclasses

import numpy as np
import pytest

import synth


def _ran_by_nodes(ctx):
    from paper_2005_09316_amd import vp
    counts, _ = vp.vp_profile_read(ctx)
    return counts[1] == 0 and counts[2] == 1


@pytest.mark.gpu
@pytest.mark.parametrize("prec,dtype,bar", [(0, 0, 1e-11), (1, 0, 1e-6)])
def test_grid_uniform_to_the_mixed_paths_tolerance_only(prec, dtype, bar):
    """Channels off a regular grid by up to 9e-13 of their frequency (alternately), which the mixed
    path's points take for regular, and baselines on which that is 3e-7 turns: the
    shapelets' phases are each channel's own."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    n = 33
    freqs = synth.channels(182e6, 80e3, n) * (1 + 4.5e-13 * np.where(np.arange(n) % 2 == 0, 1.0, -1.0))
    obs, sky = synth.make_config(1, seed=12, n_tiles=64, n_time=8, n_chan=n, n_point=1, n_gauss=0, shapelet_nmax=[20],
                                 freq_hz=freqs)
    obs = dataclasses.replace(obs, uvw_m=obs.uvw_m * 600.0, beam_fwhm_rad=0.0)
    sky.s_beta1, sky.s_beta2 = sky.s_beta1 * 0 + 1e-6, sky.s_beta2 * 0 + 1e-6
    sky.s_ra, sky.s_dec = sky.s_ra * 0 + obs.ra0 + 0.3, sky.s_dec * 0 + obs.dec0 + 0.2
    sky.p_sref = sky.p_sref * 0 + 1e-9
    ref = oracle.predict(obs, sky)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            vp.vp_profile(ctx, True)
            got = run(ctx, h.obs, h.sky, obs, prec, dtype)
            assert _ran_by_nodes(ctx)
    finally:
        vp.vp_destroy_ctx(ctx)
    F = np.abs(ref).max()
    err = np.abs(got - ref).max() / F
    phase = float(np.abs(obs.uvw_m).max() * 0.36 * freqs.max() / synth.C_LIGHT)
    print("precision", prec, "error / largest visibility %.2e, phases up to %.1e turns" % (err, phase), flush=True)
    # FP64: the phase itself is good to some 4 ulp of its turns
    assert err <= max(bar, 2 * np.pi * phase * 4 * 2.0 ** -53 if prec == 0 else 0.0)
