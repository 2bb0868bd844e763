"""Rows as correlators and flaggers leave them, at sizes that the dispatch gives to
the kernels by antenna (tests/test_antennas.py, CASES, holds sizes that go to the
vector kernels): reversed and automatic baselines, gaps, a remainder of one packed
channel, one antenna more than four blocks, and a list whose rows stop being antenna
differences at its last time, which is refused.  Predict and subtract on both paths
and types.  Bars: the paths' own, 1e-6 and 1e-11 of the total flux.

The launches of points and Gaussians show the path: two where points go by antenna,
one where both go together."""
import dataclasses

import numpy as np
import pytest

import synth

CASES = {
    # antennas, times, channels, points; share of reversed rows (the search finds antennas behind a few, not behind
    # half), automatic rows, share kept, irregular channels, moved row
    "plain": dict(n=40, n_time=14, n_chan=36, n_point=1471),
    "moved-row": dict(n=40, n_time=14, n_chan=36, n_point=1471, moved=0.5),
    "reversed": dict(n=96, n_time=4, n_chan=32, n_point=703, flip=0.04),
    "autos-packed-remainder": dict(n=32, n_time=15, n_chan=41, n_point=1489, autos=True, negative=True),
    "reversed-autos": dict(n=31, n_time=15, n_chan=42, n_point=1501, flip=0.04, autos=True),
    "reversed-gaps": dict(n=128, n_time=4, n_chan=26, n_point=240, flip=0.04, keep=0.95, negative=True),
    "reversed-irregular": dict(n=70, n_time=5, n_chan=33, n_point=609, flip=0.02, odd=True),
    "five-blocks-autos": dict(n=129, n_time=4, n_chan=64, n_point=321, autos=True, negative=True),
}
_REF = {}


def _inputs(name):
    if name not in _REF:
        import oracle
        c = dict(flip=0.0, autos=False, keep=1.0, odd=False, moved=0.0, negative=False)
        c.update(CASES[name])
        rng = np.random.default_rng(c["n"])
        freqs = synth.channels(182e6, 80e3, c["n_chan"])
        if c["odd"]:
            freqs = np.sort(np.random.default_rng(8).uniform(170e6, 190e6, c["n_chan"]))
        obs, sky = synth.make_config(1, seed=40 + c["n"], n_tiles=c["n"], n_time=c["n_time"], n_chan=c["n_chan"],
                                     n_point=c["n_point"], n_gauss=5, shapelet_nmax=[], freq_hz=freqs)
        uvw = obs.uvw_m
        if c["autos"]:  # (i, i), (i, i + 1), ... as a correlator writes them
            i, j = np.triu_indices(c["n"], k=1)
            at = np.full((c["n"], c["n"]), -1)
            at[i, j] = np.arange(i.size)
            rows = at[np.triu_indices(c["n"])]
            uvw = np.where((rows >= 0)[None, :, None], uvw[:, rows], 0.0)
        if c["keep"] < 1.0:
            uvw = uvw[:, np.sort(rng.choice(uvw.shape[1], int(c["keep"] * uvw.shape[1]), replace=False))]
        if c["flip"]:
            uvw = np.where((rng.random(uvw.shape[1]) < c["flip"])[None, :, None], -uvw, uvw)
        if c["moved"]:
            uvw = uvw.copy()
            uvw[-1, uvw.shape[1] // 2, 0] += c["moved"]
        obs = dataclasses.replace(obs, n_bl=uvw.shape[1], uvw_m=np.ascontiguousarray(uvw))
        if c["negative"]:
            sky.p_sref = np.where(np.arange(c["n_point"]) % 3 == 0, -sky.p_sref, sky.p_sref)
        _REF.clear()
        _REF[name] = obs, sky, oracle.predict(obs, sky)
    return _REF[name]


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("prec,dtype,bar", [(1, 0, 1e-6), (1, 1, 1e-6), (0, 0, 1e-11)])
def test_rows_by_antenna(name, prec, dtype, bar):
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky, ref = _inputs(name)
    data = synth.noise_c64(ref.shape, 5).astype(np.complex128)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        vp.vp_profile(ctx, True)
        for o, want in ((obs, ref), (dataclasses.replace(obs, sign=+1), np.conj(ref))):
            with Handles(ctx, o, sky) as h:
                for d in (None, data):
                    vp.vp_profile_read(ctx)
                    got = run(ctx, h.obs, h.sky, o, prec, dtype, data=d)
                    counts, _ = vp.vp_profile_read(ctx)
                    assert counts[1] == (1 if name == "moved-row" else 2), counts
                    err = oracle.error_metric(got, want if d is None else d - want, o, sky)
                    print(name, "sign", o.sign, "precision", prec, "dtype", dtype, "subtract" if d is not None else "predict",
                          "error / total flux %.2e" % err, flush=True)
                    assert err <= bar
    finally:
        vp.vp_destroy_ctx(ctx)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,bar", [(1, 1e-6), (0, 1e-6)])
def test_points_alone_into_complex64(prec, bar):
    """Without Gaussians complex64 goes straight from the kernels by antenna, on the
    FP64 path too; by time against the vector kernels' launch there is nothing to count
    but that one, so the rows are those of a case above."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky, _ = _inputs("reversed-autos")
    sky = synth.select_components(sky, gauss=[])
    ref = oracle.predict(obs, sky)
    data = synth.noise_c64(ref.shape, 6).astype(np.complex128)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            got = run(ctx, h.obs, h.sky, obs, prec, vp.VP_C64)
            res = run(ctx, h.obs, h.sky, obs, prec, vp.VP_C64, data=data)
            wide = run(ctx, h.obs, h.sky, obs, prec, vp.VP_C128)
    finally:
        vp.vp_destroy_ctx(ctx)
    e1, e2 = oracle.error_metric(got, ref, obs, sky), oracle.error_metric(res, data - ref, obs, sky)
    print("precision", prec, "error / total flux: predict %.2e, subtract %.2e" % (e1, e2), flush=True)
    assert e1 <= bar and e2 <= bar
    assert np.array_equal(got, wide.astype(np.complex64).astype(np.complex128))  # rounded once


@pytest.mark.gpu
@pytest.mark.parametrize("n_point,n_gauss,launches", [(100, 20, 1), (1500, 20, 2)])
def test_a_few_points_stay_with_the_gaussians(n_point, n_gauss, launches):
    """128 antennas, 4 times x 32 channels: what a pass by antenna costs whatever its
    points, a hundred do not bring in again (measured 49 us for 40)."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky = synth.make_config(1, seed=7, n_tiles=128, n_time=4, n_chan=32, n_point=n_point, n_gauss=n_gauss, shapelet_nmax=[],
                                 freq_hz=synth.channels(182e6, 80e3, 32))
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            vp.vp_profile(ctx, True)
            got = run(ctx, h.obs, h.sky, obs, vp.VP_PREC_MIXED, vp.VP_C64)
            counts, _ = vp.vp_profile_read(ctx)
    finally:
        vp.vp_destroy_ctx(ctx)
    assert counts[1] == launches, counts
    one = dataclasses.replace(obs, n_time=1, uvw_m=np.ascontiguousarray(obs.uvw_m[:1]))
    assert oracle.error_metric(got[:1], oracle.predict(one, sky), one, sky) <= 1e-6
