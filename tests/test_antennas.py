"""The antennas behind a list of baselines, by which point components are taken
on the matrix cores (csrc/ant_layout.h, csrc/vp_ant.hip).

On the CPU: the finder's pairs reproduce every row at every time, lists with
gaps still give the array's own antennas, rows that are no antenna differences
are refused, and the tiling covers every pair once.  On the GPU: the path
against the oracle at the edges of its blocks (32 antennas, 32 points, packed
channels), with flagged, reversed and automatic baselines, negative fluxes and
Gaussians and shapelets behind the points; test_antenna_rows_gpu.py has the sizes
at which the rule takes the path that these leave to the vector kernels.  Bars: the paths' own, 1e-6 and
1e-11 of the total flux (1e-6 for complex64)."""
import dataclasses
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def finder(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("ant") / "ant_layout_test")
    subprocess.run(["g++", "-O1", "-std=c++17", os.path.join(ROOT, "tests", "ant_layout_test.cpp"),
                    os.path.join(ROOT, "paper_2005_09316_amd", "csrc", "ant_layout.cpp"), "-o", exe], check=True)

    def run(n, keep=1.0, autos=0, order=0, jitter=0.0):
        out = subprocess.run([exe, str(n), str(keep), str(autos), str(order), str(jitter)], check=True,
                             capture_output=True, text=True).stdout.split()
        return dict(zip(("rows", "n", "bad", "dev", "channels", "uncovered"), map(float, out)))
    return run


@pytest.mark.parametrize("n", [2, 3, 31, 32, 33, 64, 65, 96, 128, 129, 160, 257])
@pytest.mark.parametrize("keep,autos", [(1.0, 0), (1.0, 1), (0.85, 0), (0.6, 1)])
@pytest.mark.parametrize("order", [0, 1])
def test_finder_on_ordered_lists(finder, n, keep, autos, order):
    r = finder(n, keep, autos, order)
    assert r["bad"] == 0 and r["uncovered"] == 0
    assert r["n"] > 0 and r["dev"] < 1e-11
    if n >= 31:  # the array's own antennas (a gap may split one)
        assert r["n"] <= n + (0 if keep == 1.0 else 3)


@pytest.mark.parametrize("n", [5, 32, 128])
def test_finder_never_gives_wrong_pairs(finder, n):
    assert finder(n, order=2)["bad"] == 0        # in no order: found or left alone
    r = finder(n, jitter=1e-6)                   # a row that moved at one time is no difference
    assert r["n"] == 0


def _case(n_tiles, n_chan, n_time, n_point, keep=None, flip=False, autos=False, negative=False, gauss=0, nmax=(), odd=False, moved=0.0):
    freqs = np.sort(np.random.default_rng(8).uniform(170e6, 190e6, n_chan)) if odd else synth.channels(182e6, 80e3, n_chan)
    obs, sky = synth.make_config(1, seed=40 + n_tiles, n_tiles=n_tiles, n_time=n_time, n_chan=n_chan, n_point=n_point,
                                 n_gauss=gauss, shapelet_nmax=list(nmax), freq_hz=freqs)
    rng = np.random.default_rng(n_tiles)
    uvw = obs.uvw_m
    if autos:
        uvw = np.concatenate([np.zeros((n_time, 1, 3)), uvw], axis=1)
    if keep is not None:
        uvw = uvw[:, np.sort(rng.choice(uvw.shape[1], int(keep * uvw.shape[1]), replace=False))]
    if flip:
        uvw = np.where((rng.random(uvw.shape[1]) < 0.5)[None, :, None], -uvw, uvw)
    if moved:  # one row that is no difference of antennas at the last time step
        uvw = uvw.copy()
        uvw[-1, uvw.shape[1] // 2, 0] += moved
    obs = dataclasses.replace(obs, n_bl=uvw.shape[1], uvw_m=np.ascontiguousarray(uvw))
    if negative:
        sky.p_sref = np.where(np.arange(n_point) % 3 == 0, -sky.p_sref, sky.p_sref)
    return obs, sky


CASES = {
    "one-block": dict(n_tiles=32, n_chan=4, n_time=1, n_point=96),
    "one-block-ragged": dict(n_tiles=21, n_chan=5, n_time=2, n_point=97),
    "two-blocks": dict(n_tiles=33, n_chan=3, n_time=1, n_point=95, keep=0.8),
    "three-blocks": dict(n_tiles=96, n_chan=2, n_time=1, n_point=96, negative=True),
    "four-blocks": dict(n_tiles=128, n_chan=1, n_time=1, n_point=200, gauss=9, nmax=[11]),
    "five-blocks": dict(n_tiles=129, n_chan=2, n_time=1, n_point=128, negative=True),
    "eight-blocks": dict(n_tiles=230, n_chan=1, n_time=1, n_point=200),
    "irregular": dict(n_tiles=70, n_chan=3, n_time=1, n_point=130, odd=True),
    "irregular-eight": dict(n_tiles=200, n_chan=2, n_time=1, n_point=210, odd=True, negative=True),
    "moved-row": dict(n_tiles=24, n_chan=3, n_time=3, n_point=400, moved=0.5),
    "flipped": dict(n_tiles=40, n_chan=3, n_time=2, n_point=150, flip=True),
    "autos": dict(n_tiles=30, n_chan=9, n_time=1, n_point=300, autos=True, gauss=5),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("prec,dtype,bar", [(1, 0, 1e-6), (1, 1, 1e-6), (0, 0, 1e-11), (0, 1, 1e-6)])
def test_points_by_antenna_match_oracle(name, prec, dtype, bar):
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    case = dict(CASES[name])
    if prec == 0:  # the FP64 kernel's rule wants more points at a few rows
        case["n_point"] += 4000 // case["n_tiles"] * 8
    obs, sky = _case(**case)
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


# Sizes that both paths' rules give to the antennas (smaller ones go to kernels
# that split rows, channels and components): blocks of 32 antennas from one to
# eight, one more and one fewer, points around multiples of 32 and 16.
BY_ANTENNA = {
    "one-block": dict(n_tiles=32, n_time=14, n_chan=40, n_point=1504),
    "one-block-ragged": dict(n_tiles=31, n_time=15, n_chan=41, n_point=1489, keep=0.97),
    "two-blocks": dict(n_tiles=40, n_time=14, n_chan=36, n_point=1471, negative=True),
    "three-blocks": dict(n_tiles=96, n_time=4, n_chan=32, n_point=703),
    "three-irregular": dict(n_tiles=70, n_time=5, n_chan=33, n_point=609, odd=True),
    "four-blocks": dict(n_tiles=128, n_time=4, n_chan=26, n_point=240, negative=True, nmax=[11]),
    "five-blocks": dict(n_tiles=129, n_time=4, n_chan=64, n_point=321),
    "eight-blocks": dict(n_tiles=230, n_time=1, n_chan=30, n_point=399, odd=True, negative=True),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(BY_ANTENNA))
@pytest.mark.parametrize("prec,dtype,bar", [(1, 0, 1e-6), (1, 1, 1e-6), (0, 0, 1e-11)])
def test_points_by_antenna_where_taken(name, prec, dtype, bar):
    """Against the oracle, and the points have a launch of their own beside the
    Gaussians'."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky = _case(gauss=5, **BY_ANTENNA[name])
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
    print(name, "precision", prec, "dtype", dtype, "error / total flux %.2e" % err, flush=True)
    assert counts[1] == 2, counts
    assert err <= bar


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(n_tiles=128, n_chan=4, n_time=4, n_point=3000),
                                dict(n_tiles=40, n_chan=32, n_time=4, n_point=2000, odd=True),
                                dict(n_tiles=128, n_chan=26, n_time=4, n_point=3000),
                                dict(n_tiles=40, n_chan=40, n_time=14, n_point=2000, odd=True)],
                         ids=["128", "40-irregular", "128-by-antenna", "40-by-antenna-irregular"])
def test_fp64_points_against_80_bits(kw):
    """The FP64 path on sampled rows, against numpy's extended precision.  A
    point's phase is good to the rounding of its direction (4 ulp of each of l,
    m, n - 1), of the row and of the antennas fitted to rows (3 ulp of the row);
    amplitudes, factors, products and sums to 16 ulp of the total flux."""
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky = _case(**kw)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            got = np.asarray(run(ctx, h.obs, h.sky, obs, vp.VP_PREC_FP64, vp.VP_C128)).reshape(-1, obs.n_chan)
    finally:
        vp.vp_destroy_ctx(ctx)
    rows = np.random.default_rng(3).choice(got.shape[0], 40, replace=False)
    L = np.longdouble
    two_pi = 2 * L("3.14159265358979323846264338327950288")
    uvw, ra, dec = obs.uvw_m.reshape(-1, 3)[rows].astype(L), sky.p_ra.astype(L), sky.p_dec.astype(L)
    s0, c0, da = np.sin(L(obs.dec0)), np.cos(L(obs.dec0)), ra - L(obs.ra0)
    lmn = np.stack([np.cos(dec) * np.sin(da), np.sin(dec) * c0 - np.cos(dec) * s0 * np.cos(da),
                    np.sin(dec) * s0 + np.cos(dec) * c0 * np.cos(da) - 1])
    turns = uvw @ lmn
    ulp = 2.0 ** -53
    for k in range(obs.n_chan):
        fk = L(obs.freq_hz[k]) / L(synth.C_LIGHT)
        flux = sky.p_sref.astype(L) * (L(obs.freq_hz[k]) / L(sky.nu_ref_hz)) ** sky.p_alpha.astype(L)
        th = L(obs.beam_fwhm_rad) * L(obs.beam_nu_ref_hz) / L(obs.freq_hz[k])
        flux *= np.exp(-4 * np.log(L(2)) * (np.arcsin(np.hypot(lmn[0], lmn[1])) / th) ** 2)
        ph = two_pi * (turns * fk - np.rint(turns * fk))
        ref = (np.cos(ph) + 1j * obs.sign * np.sin(ph)) @ flux
        bar = float(two_pi * fk) * 7 * ulp * (np.abs(uvw) @ np.abs(lmn) @ np.abs(flux)).astype(float) + 16 * ulp * float(np.abs(flux).sum())
        err = np.abs((got[rows, k].astype(np.clongdouble) - ref).astype(complex))
        assert (err <= bar).all(), (k, float((err / bar).max()))
