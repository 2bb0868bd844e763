"""Skies that lie wholly in the skirts of the primary beam, so that what reaches
the data is 1e-5 to 1e-30 of the catalogue's fluxes.  The bars are the paths' own,
1e-6 and 1e-11 of the apparent total flux (beam included), at every distance from
the beam's centre."""
import dataclasses
import math

import numpy as np
import pytest

import synth

BARS = {1: 1e-6, 0: 1e-11}


def _sky(obs, n_point, n_gauss, rho, radius, seed=1, steep=None):
    """Components within `radius` of a direction `rho` (radians) north of the phase centre."""
    rng = np.random.default_rng(seed)
    _, sky = synth.make_config(1, seed=seed, n_tiles=4, n_time=1, n_chan=4, n_point=n_point, n_gauss=n_gauss,
                               shapelet_nmax=[])
    for n, ra, dec in ((n_point, "p_ra", "p_dec"), (n_gauss, "g_ra", "g_dec")):
        r, th = radius * np.sqrt(rng.random(n)), 2 * np.pi * rng.random(n)
        setattr(sky, dec, obs.dec0 + rho + r * np.sin(th))
        setattr(sky, ra, obs.ra0 + r * np.cos(th) / np.cos(obs.dec0 + rho))
    if steep is not None:
        sky.p_alpha = np.full(n_point, steep)
    return sky


def _obs(n_tiles, n_time, n_chan, fwhm_deg, **kw):
    obs, _ = synth.make_config(1, seed=60 + n_tiles, n_tiles=n_tiles, n_time=n_time, n_chan=n_chan, n_point=1, n_gauss=0,
                               shapelet_nmax=[], **kw)
    return dataclasses.replace(obs, beam_fwhm_rad=math.radians(fwhm_deg), beam_nu_ref_hz=float(np.mean(obs.freq_hz)))


@pytest.mark.gpu
@pytest.mark.parametrize("fwhms", [0.0, 2.0, 3.0, 3.5, 4.0, 5.0])
@pytest.mark.parametrize("prec,dtype", [(1, 0), (1, 1), (0, 0)])
def test_points_by_antenna_in_the_skirts(fwhms, prec, dtype):
    """Points alone have two launches beside Gaussians: they were taken by antenna."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs = _obs(128, 4, 26, 5.0)
    sky = _sky(obs, 1500, 3, math.radians(5.0) * fwhms, math.radians(0.25))
    ref = oracle.predict(obs, sky)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            vp.vp_profile(ctx, True)
            vp.vp_profile_read(ctx)
            got = run(ctx, h.obs, h.sky, obs, prec, dtype)
            counts, _ = vp.vp_profile_read(ctx)
    finally:
        vp.vp_destroy_ctx(ctx)
    err = oracle.error_metric(got, ref, obs, sky)
    print(fwhms, "FWHM, precision", prec, "dtype", dtype, "error / apparent flux %.2e" % err, flush=True)
    assert counts[1] == 2, counts
    assert err <= BARS[prec]


@pytest.mark.gpu
def test_points_by_antenna_far_below_the_reference_frequency_flux():
    """A spectrum that leaves 2^-18 of S_ref in the band: the amplitudes are
    scaled by what is there."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs = _obs(128, 4, 26, 25.0)
    sky = _sky(obs, 1500, 0, 0.0, math.radians(2.0), steep=-6.0)
    sky.nu_ref_hz = float(obs.freq_hz[0]) / 8.0
    ref = oracle.predict(obs, sky)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            got = run(ctx, h.obs, h.sky, obs, 1, 0)
    finally:
        vp.vp_destroy_ctx(ctx)
    err = oracle.error_metric(got, ref, obs, sky)
    print("error / total flux %.2e" % err, flush=True)
    assert err <= 1e-6
