"""Points and Gaussians by nodes (csrc/shp_nodes.h, pg_nodes; k_pg_nodes): on
the CPU, the number of Chebyshev nodes that the library takes for a field and a
band suffices for every phase, spectral index and envelope within its bounds; on
the GPU, points and Gaussians against the oracle: node counts around the waves'
shares, channels around multiples of 16, rows around the workgroup's, few
components, a sky beside the phase centre and across the origin of right ascension,
irregular and reversed channels.  The smallest of these go to the kernels by channels
(csrc/dispatch.h, whose lines test_dispatch.py holds).  Bars: the paths' own, 1e-6 and
1e-11 of the total flux (1e-6 for complex64)."""
import dataclasses
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def node_count(tmp_path_factory):
    d = tmp_path_factory.mktemp("pg")
    src = d / "n.cpp"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "%s"\n'
                   'int main(int c, char **v) { for (int i = 1; i + 3 < c; i += 4) '
                   'printf("%%d\\n", vp::pg_nodes(atof(v[i]), atof(v[i + 1]), atof(v[i + 2]), atof(v[i + 3]))); }\n'
                   % os.path.join(ROOT, "paper_2005_09316_amd", "csrc", "shp_nodes.h"))
    exe = str(d / "n")
    subprocess.run(["g++", "-O1", "-std=c++17", str(src), "-o", exe], check=True)

    def run(args):
        out = subprocess.run([exe] + [repr(float(x)) for a in args for x in a], check=True, capture_output=True, text=True)
        return [int(x) for x in out.stdout.split()]
    return run


@pytest.mark.parametrize("tol", [1e-6, 1e-10, 1e-12])
def test_enough_nodes_for_every_component(node_count, tol):
    """Interpolation on [-1, 1] of (1 + delta z)^alpha 2^(-Q (1 + delta z)^2)
    e^(i t z), |t| <= w, |alpha| <= amax, Q from 0 to where the envelope has
    vanished: the error stays below the tolerance (and 2e-13, the rounding of
    the interpolation itself)."""
    cases = [(w, d, am, tol) for w in (0.0, 0.3, 2.0, 5.5, 9.0, 20.0, 30.0) for d in (1e-4, 0.02, 0.09, 0.3, 0.5)
             for am in (0.0, 0.8, 3.0)]
    z = np.linspace(-1, 1, 301) + 1e-9
    took = 0
    for (w, d, am, _), M in zip(cases, node_count(cases)):
        if M == 0:
            continue
        took += 1
        k = np.arange(M)
        zn = np.cos(np.pi * (2 * k + 1) / (2 * M))
        wt = (-1.0) ** k * np.sin(np.pi * (2 * k + 1) / (2 * M))
        L = wt / (z[:, None] - zn)
        L /= L.sum(1, keepdims=True)
        for t in (w, -w, 0.6 * w):
            for al in (am, -am):
                for Q in (0.0, 0.1, 1.0, 5.0, 20.0, 60.0):
                    def f(x):
                        return (1 + d * x) ** al * 2.0 ** (-Q * (1 + d * x) ** 2) * np.exp(1j * t * x)
                    err = np.abs(L @ f(zn) - f(z)).max()
                    assert err <= tol + 2e-13, (w, d, am, t, al, Q, M, err)
    assert took > 40


def test_refuses_what_it_does_not_cover(node_count):
    bad = [(50.0, 0.1, 1.0, 1e-10), (float("nan"), 0.1, 1.0, 1e-10), (float("inf"), 0.1, 1.0, 1e-10),
           (2.0, float("nan"), 1.0, 1e-10), (2.0, 0.1, float("inf"), 1e-10), (2.0, 0.1, 1e4, 1e-10), (2.0, 2.0, 1.0, 1e-10)]
    assert node_count(bad) == [0] * len(bad)


def _case(n_tiles, n_time, n_chan, n_point, n_gauss, radius, d_ra=0.0, d_dec=0.0, wrap=False, odd=False, reverse=False,
          nmax=(), beam=True, width=None, ragged=0):
    freqs = synth.channels(182e6, (width or 10e6) / n_chan, n_chan)
    if odd:
        freqs = np.sort(np.random.default_rng(8).uniform(freqs[0], freqs[-1], n_chan))
    if reverse:
        freqs = freqs[::-1].copy()
    obs, sky = synth.make_config(1, seed=90 + n_tiles, n_tiles=n_tiles, n_time=n_time, n_chan=n_chan, n_point=n_point,
                                 n_gauss=n_gauss, shapelet_nmax=list(nmax), freq_hz=freqs)
    if ragged:
        obs = dataclasses.replace(obs, n_bl=obs.n_bl - ragged, uvw_m=np.ascontiguousarray(obs.uvw_m[:, ragged:]))
    rng = np.random.default_rng(n_tiles + n_chan)
    ra0 = 0.0 if wrap else 1.3
    for n, ra, dec in ((n_point, "p_ra", "p_dec"), (n_gauss, "g_ra", "g_dec")):
        r, th = radius * np.sqrt(rng.random(n)), 2 * np.pi * rng.random(n)
        setattr(sky, dec, obs.dec0 + d_dec + r * np.sin(th))
        setattr(sky, ra, np.mod(ra0 + d_ra + r * np.cos(th) / np.cos(obs.dec0), 2 * np.pi))
    return dataclasses.replace(obs, ra0=ra0, beam_fwhm_rad=obs.beam_fwhm_rad if beam else 0.0), sky


CASES = {
    "points": dict(n_tiles=12, n_time=1, n_chan=48, n_point=70, n_gauss=0, radius=0.002),
    "gauss": dict(n_tiles=13, n_time=2, n_chan=65, n_point=0, n_gauss=70, radius=0.004),
    "one-each": dict(n_tiles=5, n_time=1, n_chan=33, n_point=1, n_gauss=1, radius=0.003),
    "few-channels": dict(n_tiles=24, n_time=1, n_chan=36, n_point=200, n_gauss=9, radius=1e-4),
    "by-antenna-and-nodes": dict(n_tiles=64, n_time=2, n_chan=96, n_point=1500, n_gauss=65, radius=0.003),
    "ragged-rows": dict(n_tiles=20, n_time=3, n_chan=79, n_point=129, n_gauss=63, radius=0.004, ragged=7),
    "off-centre": dict(n_tiles=17, n_time=1, n_chan=128, n_point=80, n_gauss=40, radius=0.001, d_ra=0.006, d_dec=-0.004),
    "across-zero": dict(n_tiles=17, n_time=1, n_chan=128, n_point=80, n_gauss=40, radius=0.004, wrap=True),
    "many-nodes": dict(n_tiles=16, n_time=1, n_chan=200, n_point=90, n_gauss=30, radius=0.01, width=30e6),
    "irregular": dict(n_tiles=19, n_time=1, n_chan=90, n_point=100, n_gauss=30, radius=0.003, odd=True, beam=False),
    "reversed-shapelet": dict(n_tiles=19, n_time=1, n_chan=90, n_point=100, n_gauss=30, radius=0.003, reverse=True, nmax=[9], wrap=True),
    "wide": dict(n_tiles=12, n_time=1, n_chan=40, n_point=70, n_gauss=30, radius=0.2),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("prec,dtype,bar", [(1, 0, 1e-6), (1, 1, 1e-6), (0, 0, 1e-11), (0, 1, 1e-6)])
def test_points_and_gaussians_by_nodes_match_oracle(name, prec, dtype, bar):
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky = _case(**CASES[name])
    ref = oracle.predict(obs, sky)
    data = synth.noise_c64(ref.shape, 5).astype(np.complex128)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            got = run(ctx, h.obs, h.sky, obs, prec, dtype)
            res = run(ctx, h.obs, h.sky, obs, prec, dtype, data=data)
    finally:
        vp.vp_destroy_ctx(ctx)
    e1, e2 = oracle.error_metric(got, ref, obs, sky), oracle.error_metric(res, data - ref, obs, sky)
    print(name, "precision", prec, "dtype", dtype, "error / total flux: predict %.2e, subtract %.2e" % (e1, e2), flush=True)
    assert e1 <= bar and e2 <= bar


# Observations of a few tiles, whose components are split over waves and lanes:
# (tiles, times, channels, points, Gaussians); 256 rows x 8 channels are a tile,
# and the kernels change at 4, 40 and 64 of them.
SMALL = [(5, 1, 3, 3, 2), (24, 1, 31, 1, 0), (40, 1, 7, 63, 64), (30, 1, 100, 17, 130), (40, 2, 50, 17, 47),
         (60, 2, 33, 0, 65), (90, 2, 41, 63, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("size", SMALL, ids=["-".join(map(str, s)) for s in SMALL])
@pytest.mark.parametrize("prec,dtype,bar", [(1, 0, 1e-6), (1, 1, 1e-6), (0, 0, 1e-11), (0, 1, 1e-6)])
def test_small_observations_match_oracle(size, prec, dtype, bar):
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    ctx = vp.vp_create_ctx(0, 0)
    try:
        for odd in (False, True):
            obs, sky = _case(*size, radius=0.2, odd=odd, wrap=True, nmax=[12])
            ref = oracle.predict(obs, sky)
            data = synth.noise_c64(ref.shape, 5).astype(np.complex128)
            with Handles(ctx, obs, sky) as h:
                got = run(ctx, h.obs, h.sky, obs, prec, dtype)
                res = run(ctx, h.obs, h.sky, obs, prec, dtype, data=data)
            e1, e2 = oracle.error_metric(got, ref, obs, sky), oracle.error_metric(res, data - ref, obs, sky)
            print(size, odd, "precision", prec, "dtype", dtype, "error / total flux %.2e %.2e" % (e1, e2), flush=True)
            assert e1 <= bar and e2 <= bar
    finally:
        vp.vp_destroy_ctx(ctx)
