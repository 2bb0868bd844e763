"""The antennas behind a list of baselines, by which point components are taken
on the matrix cores (csrc/ant_layout.h, csrc/vp_ant.hip).

On the CPU: the finder's pairs reproduce every row at every time, lists with
gaps still give the array's own antennas, rows that are no antenna differences
are refused, and the tiling covers every pair once.  On the GPU: the path
against the oracle at the edges of its blocks (32 antennas, 32 points, packed
channels), with flagged, reversed and automatic baselines, negative fluxes and
Gaussians and shapelets behind the points.  Bar: the mixed path's, 1e-6 of the
total flux."""
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


def _case(n_tiles, n_chan, n_time, n_point, keep=None, flip=False, autos=False, negative=False, gauss=0, nmax=(), odd=False):
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
    "flipped": dict(n_tiles=40, n_chan=3, n_time=2, n_point=150, flip=True),
    "autos": dict(n_tiles=30, n_chan=9, n_time=1, n_point=300, autos=True, gauss=5),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("dtype", [0, 1])
def test_points_by_antenna_match_oracle(name, dtype):
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky = _case(**CASES[name])
    ref = oracle.predict(obs, sky)
    data = synth.noise_c64(ref.shape, 5).astype(np.complex128)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            got = run(ctx, h.obs, h.sky, obs, vp.VP_PREC_MIXED, dtype)
            res = run(ctx, h.obs, h.sky, obs, vp.VP_PREC_MIXED, dtype, data=data)
    finally:
        vp.vp_destroy_ctx(ctx)
    e1, e2 = oracle.error_metric(got, ref, obs, sky), oracle.error_metric(res, data - ref, obs, sky)
    print(name, "dtype", dtype, "error / total flux: predict %.2e, subtract %.2e" % (e1, e2), flush=True)
    assert e1 <= 1e-6 and e2 <= 1e-6
