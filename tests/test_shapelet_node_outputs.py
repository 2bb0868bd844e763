"""Shapelets at sizes that the dispatch gives to the node kernels (k_shp_nodes,
k_shp_nodes64; tests/test_shapelet_nodes.py holds sizes that go to the channel
kernels).  Up to four points beside shapelets go along with the node kernels'
outputs, without a launch of their own: that the points' launch count is 0 shows
which kernel ran.  Bars: the paths' own, 1e-6 and 1e-11 (1e-6 for complex64), of the
total flux or of the largest visibility where that is larger (coefficients drawn at
random may cancel at the centre and not elsewhere: up to 17 times the flux here,
where the kernels by channels err by as much, 1.1e-6 of the flux)."""
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


CASES = {
    # name: (tiles, times, orders, spectral terms, frequencies); rows x channels are over 512 workgroups of the
    # channel kernels on both paths (256 rows x 1 channel mixed, x 4 FP64)
    "narrow-16": (64, 17, [30, 7], 1, synth.channels(182e6, 80e3, 16)),
    "narrow-17-terms": (63, 14, [30], 2, synth.channels(182e6, 80e3, 17)),
    "wide-96": (40, 8, [96, 0, 40], 1, synth.band(150e6, 180e6, 96)),
    "wide-45": (60, 7, [54], 1, synth.band(150e6, 180e6, 45)),
    "many-shapelets": (44, 9, [63, 11, 40, 31, 20, 33, 8, 32, 1, 52], 1, synth.band(160e6, 180e6, 64)),
    "irregular": (61, 8, [47, 21], 1, np.sort(np.random.default_rng(3).uniform(170e6, 190e6, 37))),
    "irregular-reversed": (61, 8, [33], 1, np.sort(np.random.default_rng(4).uniform(170e6, 190e6, 39))[::-1].copy()),
    # the middle channel is the middle of the band: a node where their number is odd
    "on-a-node": (61, 9, [22], 1, synth.channels(182e6, 500e3, 33)),
}
_REF = {}


def _inputs(name):
    """Observation (ragged in its rows), shapelets alone, five points alone, and the oracle's visibilities of each."""
    if name not in _REF:
        import oracle
        tiles, times, orders, terms, freqs = CASES[name]
        obs, sky = synth.make_config(1, seed=77, n_tiles=tiles, n_time=times, n_chan=len(freqs), n_point=5, n_gauss=0,
                                     shapelet_nmax=orders, freq_hz=freqs)
        obs = dataclasses.replace(obs, n_bl=obs.n_bl - 5, uvw_m=np.ascontiguousarray(obs.uvw_m[:, 5:]))
        if terms > 1:
            sky = synth.with_spectral_terms(sky, np.random.default_rng(4), terms)
        only = synth.select_components(sky, points=[], gauss=[])
        refs = [oracle.predict(obs, only)] + [oracle.predict(obs, synth.select_components(sky, points=list(range(n)), shapelets=[]))
                                              for n in (1, 4, 5)]
        _REF.clear()
        _REF[name] = obs, sky, refs
    return _REF[name]


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("prec,dtype,bar", [(0, 0, 1e-11), (1, 0, 1e-6), (1, 1, 1e-6), (0, 1, 1e-6)])
def test_shapelets_by_nodes(name, prec, dtype, bar):
    """Alone (both signs of the exponent, predict and subtract), with one and four
    points that go along, and with five that do not."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky, (shp, *points) = _inputs(name)
    plus = dataclasses.replace(obs, sign=+1)
    data = synth.noise_c64(shp.shape, 5).astype(np.complex128)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        vp.vp_profile(ctx, True)
        for n, pts in ((1, points[0]), (4, points[1]), (5, points[2]), (0, 0.0)):
            part = synth.select_components(sky, points=list(range(n)))
            for o, ref in ((obs, shp + pts), (plus, np.conj(shp + pts))):
                with Handles(ctx, o, part) as h:
                    got = run(ctx, h.obs, h.sky, o, prec, dtype)
                    counts, _ = vp.vp_profile_read(ctx)
                    # the path: a plan of the pair's shapelets and band alone, the same for all four skies
                    assert counts[1] == (1 if n == 5 else 0) and counts[2] == 1, (n, counts)
                    res = run(ctx, h.obs, h.sky, o, prec, dtype, data=data)
                    vp.vp_profile_read(ctx)
                assert np.all(np.isfinite(got))
                F = np.maximum(oracle.total_flux(o, part), np.abs(ref).max(axis=(0, 1)))
                e1, e2 = (np.abs(got - ref) / F).max(), (np.abs(res - (data - ref)) / F).max()
                print(name, n, "points, sign", o.sign, "precision", prec, "dtype", dtype,
                      "error: predict %.2e, subtract %.2e" % (e1, e2), flush=True)
                assert e1 <= bar and e2 <= bar
    finally:
        vp.vp_destroy_ctx(ctx)
