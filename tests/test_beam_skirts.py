"""Skies that lie wholly in the skirts of the primary beam, so that what reaches
the data is 1e-5 to 1e-30 of the catalogue's fluxes.  The bars are the paths' own,
1e-6 and 1e-11 of the apparent total flux (beam included), at every distance from
the beam's centre."""
import dataclasses
import math
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
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


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("pgbeam")
    src = d / "n.cpp"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "%s"\n'
                   'int main(int c, char **v) { for (int i = 1; i + 4 < c; i += 5) { double a[5]; '
                   'for (int j = 0; j < 5; ++j) a[j] = atof(v[i + j]); '
                   'printf("%%d %%.17g\\n", vp::pg_nodes(a[0], a[1], a[2], a[3], a[4]), vp::pg_spread(a[1], a[2], a[4])); } }\n'
                   % os.path.join(ROOT, "paper_2005_09316_amd", "csrc", "shp_nodes.h"))
    exe = str(d / "n")
    subprocess.run(["g++", "-O1", "-std=c++17", str(src), "-o", exe], check=True)

    def run(args):
        out = subprocess.run([exe] + [repr(float(x)) for a in args for x in a], check=True, capture_output=True,
                             text=True).stdout.split()
        return [(int(m), float(s)) for m, s in zip(out[::2], out[1::2])]
    return run


@pytest.mark.parametrize("tol", [1e-6, 1e-10, 1e-12])
def test_enough_nodes_under_a_beam(rule, tol):
    """As for every component without one: the interpolation's error over the
    flux that beam and spectrum leave at the channel stays below the tolerance
    (and 2e-13, its rounding, times the flux's spread over the band)."""
    cases = [(w, d, am, tol, A) for w in (0.0, 0.5, 3.0, 9.0, 20.0) for d in (1e-4, 0.02, 0.09, 0.15, 0.3)
             for am in (0.0, 0.8, 3.0) for A in (0.0, 0.7, 2.8, 11.1, 25.0, 44.4)]
    z = np.linspace(-1, 1, 301) * (1 - 1e-9)
    took = 0
    for (w, d, am, _, A), (M, spread) in zip(cases, rule(cases)):
        if M == 0:
            continue
        took += 1
        k = np.arange(M)
        zn = np.cos(np.pi * (2 * k + 1) / (2 * M))
        wt = (-1.0) ** k * np.sin(np.pi * (2 * k + 1) / (2 * M))
        L = wt / (z[:, None] - zn)
        L /= L.sum(1, keepdims=True)
        for t in (w, -w):
            for al in (am, -am):
                def S(x):
                    return (1 + d * x) ** al * np.exp(-A * ((1 + d * x) ** 2 - 1))
                assert np.log(S(z).max() / S(z).min()) <= spread + 1e-9
                for Q in (0.0, 1.0, 20.0):
                    def f(x):
                        return S(x) * 2.0 ** (-Q * (1 + d * x) ** 2) * np.exp(1j * t * x)
                    err = (np.abs(L @ f(zn) - f(z)) / S(z)).max()
                    assert err <= tol + 2e-13 * np.exp(spread), (w, d, am, A, t, al, Q, M, err)
    assert took > 100


@pytest.mark.gpu
@pytest.mark.parametrize("fwhms", [0.0, 1.0, 2.0, 3.0, 4.0])
@pytest.mark.parametrize("prec,dtype", [(1, 0), (0, 0)])
def test_narrow_fields_in_the_skirts(fwhms, prec, dtype):
    """A small array, a dish's beam and a band of 18%: near the centre the sums go
    by nodes, further out the spread of the beam over the band forbids it."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    rng = np.random.default_rng(5)
    freqs = synth.band(165e6, 199e6, 100)
    fwhm = math.radians(0.5)
    obs = synth.make_obs(rng, 16, 1, freqs, radius_m=50.0, beam_fwhm_rad=fwhm, beam_nu_ref_hz=182e6)
    sky = _sky(obs, 50, 20, fwhm * fwhms, fwhm / 20)
    ref = oracle.predict(obs, sky)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            got = run(ctx, h.obs, h.sky, obs, prec, dtype)
    finally:
        vp.vp_destroy_ctx(ctx)
    err = oracle.error_metric(got, ref, obs, sky)
    print(fwhms, "FWHM, precision", prec, "error / apparent flux %.2e" % err, flush=True)
    assert err <= BARS[prec]
