"""The rules by which a call's kernels are chosen (csrc/dispatch.h), evaluated on the
CPU at sizes whose two sides were measured, and on the GPU the kernels at sizes that
the rules give to them."""
import dataclasses
import math
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rule(name, *arguments): the rule's answer (nodes, or 0 and 1)."""
    d = tmp_path_factory.mktemp("dispatch")
    src = d / "d.cpp"
    src.write_text('''#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "%s"
int main(int c, char **v) {
  double a[16];
  for (int i = 2; i < c && i < 18; ++i) a[i - 2] = atof(v[i]);
  int r = -1;
  if (!strcmp(v[1], "shapelets"))  // f64 S N f_lo f_hi rows K
    r = vp::shp_plan_nodes(a[0], a[1], a[2], a[1] * vp::shp_size(a[0] ? vp::kFP64 : vp::kMixed, a[2]), a[3], a[4], a[5], a[6]);
  if (!strcmp(v[1], "points"))  // f64 P G apart b_max amax f_lo f_hi fwhm nu_ref rows K uniform
    r = vp::pg_plan_nodes(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12]);
  if (!strcmp(v[1], "split")) r = vp::pg_split(a[0], a[1], a[2], a[3]);  // f64 tiles P G
  if (!strcmp(v[1], "small")) r = vp::pg_small(a[0], a[1], a[2], a[3]);  // f64 tiles n uniform
  printf("%%d", r);
}
''' % os.path.join(ROOT, "paper_2005_09316_amd", "csrc", "dispatch.h"))
    exe = str(d / "d")
    subprocess.run(["g++", "-O1", "-std=c++17", str(src), "-o", exe], check=True)

    def run(name, *args):
        return int(subprocess.run([exe, name] + [repr(float(x)) for x in args], check=True, capture_output=True, text=True).stdout)
    return run


def _band(chans, width=80e3):
    f = synth.channels(182e6, width, chans)
    return f[0], f[-1]


# (f64, shapelets, order, rows, channels, by nodes): us by nodes and by channels as measured
SHAPELETS = [
    (1, 20, 40, 32512, 20, False),   # 1800, 1000
    (1, 28, 20, 32512, 64, False),   # 2120, 1460
    (1, 16, 70, 32512, 20, False),   # 2650, 1970
    (1, 5, 40, 32512, 20, True),     # 187, 261
    (1, 20, 20, 32512, 64, True),    # 836, 1047
    (0, 45, 20, 32512, 12, False),   # 2.2 times the channels'
    (0, 60, 70, 32512, 12, False),   # 1.8 times
    (0, 28, 20, 32512, 20, True),    # 449, 617
    (0, 10, 70, 32512, 64, True),    # 632, 1817
]


@pytest.mark.parametrize("case", SHAPELETS, ids=["-".join(map(str, c[:5])) for c in SHAPELETS])
def test_shapelets_by_the_faster_kernel(rule, case):
    f64, S, N, rows, K, nodes = case
    assert (rule("shapelets", f64, S, N, *_band(K), rows, K) > 0) == nodes


@pytest.mark.gpu
@pytest.mark.parametrize("S,nodes", [(3, True), (20, False)])
def test_many_shapelets_in_fp64(rule, S, nodes):
    """The point that goes along with the outputs by nodes has a launch of its own by
    channels.  Against the oracle at the first time."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    obs, sky = synth.make_config(1, seed=3, n_tiles=64, n_time=12, n_chan=24, n_point=1, n_gauss=0,
                                 shapelet_nmax=[20, 17, 24, 9] * 5, freq_hz=synth.channels(182e6, 80e3, 24))
    sky = synth.select_components(sky, shapelets=list(range(S)))
    assert (rule("shapelets", 1, S, 24, *_band(24), obs.n_time * obs.n_bl, 24) > 0) == nodes
    ctx = vp.vp_create_ctx(0, 0)
    try:
        vp.vp_profile(ctx, True)
        with Handles(ctx, obs, sky) as h:
            got = run(ctx, h.obs, h.sky, obs, vp.VP_PREC_FP64, vp.VP_C128)
            counts, _ = vp.vp_profile_read(ctx)
    finally:
        vp.vp_destroy_ctx(ctx)
    assert counts[1] == (0 if nodes else 1) and counts[2] == 1, counts
    one = dataclasses.replace(obs, n_time=1, uvw_m=np.ascontiguousarray(obs.uvw_m[:1]))
    ref = oracle.predict(one, sky)
    F = np.maximum(oracle.total_flux(one, sky), np.abs(ref).max(axis=(0, 1)))
    err = (np.abs(got[:1] - ref) / F).max()
    print(S, "shapelets, error %.2e" % err, flush=True)
    assert err <= 1e-11


# (f64, points, Gaussians, rows, channels, field radius, by nodes): us by nodes and by channels as measured
POINTS = [
    (0, 1, 0, 2016, 384, 0.01, False),      # 16.6, 9.7
    (1, 1, 0, 2016, 384, 0.01, False),      # 20.5, 11.5
    (0, 8, 0, 2016, 384, 0.001, False),     # 15.2, 11.1
    (1, 30, 10, 32512, 64, 0.009, False),   # 113, 68
    (1, 60, 0, 8128, 64, 0.009, False),     # 31.8, 29.2
    (0, 0, 300, 8128, 384, 0.003, True),
    (0, 4540, 1791, 32512, 384, 0.009, True),  # 2900, 9000
    (1, 4540, 1791, 32512, 384, 0.009, True),
]


@pytest.mark.parametrize("case", POINTS, ids=["-".join(map(str, c[:5])) for c in POINTS])
def test_points_by_the_faster_kernel(rule, case):
    f64, P, G, rows, K, radius, nodes = case
    assert (rule("points", f64, P, G, radius, 3000.0, 1.0, *_band(K), 0.0, 0.0, rows, K, 1) > 0) == nodes


def _pg_rule(rule, f64, obs, sky):
    """The rule for a pair, from the bounds that creating them takes."""
    ra, dec = np.concatenate([sky.p_ra, sky.g_ra]), np.concatenate([sky.p_dec, sky.g_dec])
    x = np.mod(ra - ra[0] + np.pi, 2 * np.pi) - np.pi
    mra, mdec = ra[0] + 0.5 * (x.min() + x.max()), 0.5 * (dec.min() + dec.max())
    da, dd, c = np.mod(ra - mra + np.pi, 2 * np.pi) - np.pi, np.abs(dec - mdec), abs(math.cos(mdec))
    reach = math.sqrt((dd * dd + c * (c + dd) * da * da).max())
    sd, sa = math.sin(0.5 * (mdec - obs.dec0)), math.sin(0.5 * (mra - obs.ra0))
    to_mid = 2 * math.sqrt(sd * sd + abs(math.cos(mdec) * math.cos(obs.dec0)) * sa * sa)
    b_max = math.sqrt((obs.uvw_m ** 2).sum(axis=-1).max())
    fk = obs.freq_hz / synth.C_LIGHT
    dev = np.abs(fk - (fk[0] + np.arange(fk.size) * (fk[-1] - fk[0]) / (fk.size - 1))).max() / fk[0]
    amax = np.abs(np.concatenate([sky.p_alpha, sky.g_alpha])).max()
    return rule("points", f64, sky.n_point, sky.n_gauss, min(2.0, to_mid + reach), b_max, amax, obs.freq_hz.min(),
                obs.freq_hz.max(), obs.beam_fwhm_rad, obs.beam_nu_ref_hz, obs.n_time * obs.n_bl, obs.n_chan,
                dev <= (1e-15 if f64 else 1e-12))


# The edges of k_pg_nodes at component counts that send both paths there: node counts around the waves' shares,
# channels around multiples of 16, rows around the workgroup's, a sky beside the centre, across the origin of right
# ascension, irregular and reversed channels, points by antenna beside, shapelets by nodes behind.
BY_NODES = {
    "points": dict(n_tiles=64, n_time=5, n_chan=96, n_point=150, n_gauss=0, radius=0.002),
    "gauss": dict(n_tiles=65, n_time=5, n_chan=129, n_point=0, n_gauss=130, radius=0.003),
    "one-chunk": dict(n_tiles=64, n_time=5, n_chan=200, n_point=64, n_gauss=0, radius=0.002, width=4e6),
    "few-nodes": dict(n_tiles=64, n_time=6, n_chan=72, n_point=100, n_gauss=65, radius=1e-4),
    "ragged-rows": dict(n_tiles=61, n_time=7, n_chan=143, n_point=121, n_gauss=127, radius=0.003, ragged=7),
    "off-centre": dict(n_tiles=64, n_time=5, n_chan=160, n_point=80, n_gauss=140, radius=0.001, d_ra=0.004, d_dec=-0.003),
    "across-zero": dict(n_tiles=64, n_time=5, n_chan=160, n_point=80, n_gauss=140, radius=0.003, wrap=True),
    "many-nodes": dict(n_tiles=64, n_time=5, n_chan=300, n_point=100, n_gauss=130, radius=0.008, width=30e6),
    "irregular": dict(n_tiles=63, n_time=5, n_chan=90, n_point=100, n_gauss=90, radius=0.003, odd=True, beam=False),
    "reversed-shapelet": dict(n_tiles=64, n_time=5, n_chan=120, n_point=100, n_gauss=130, radius=0.002, reverse=True,
                              nmax=[9], wrap=True),
    "antennas-beside": dict(n_tiles=64, n_time=6, n_chan=96, n_point=900, n_gauss=165, radius=0.003),
}
_REF = {}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(BY_NODES))
@pytest.mark.parametrize("prec,dtype,bar", [(1, 0, 1e-6), (1, 1, 1e-6), (0, 0, 1e-11), (0, 1, 1e-6)])
def test_points_and_gaussians_where_by_nodes(rule, name, prec, dtype, bar):
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    from tests.test_pg_nodes import _case
    if name not in _REF:
        _REF.clear()
        obs, sky = _case(**BY_NODES[name])
        _REF[name] = obs, sky, oracle.predict(obs, sky)
    obs, sky, ref = _REF[name]
    assert _pg_rule(rule, 1 - prec, obs, sky) > 0
    data = synth.noise_c64(ref.shape, 5).astype(np.complex128)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            got = run(ctx, h.obs, h.sky, obs, prec, dtype)
            res = run(ctx, h.obs, h.sky, obs, prec, dtype, data=data)
    finally:
        vp.vp_destroy_ctx(ctx)
    F = np.maximum(oracle.total_flux(obs, sky), np.abs(ref).max(axis=(0, 1)))
    e1, e2 = (np.abs(got - ref) / F).max(), (np.abs(res - (data - ref)) / F).max()
    print(name, "precision", prec, "dtype", dtype, "error: predict %.2e, subtract %.2e" % (e1, e2), flush=True)
    assert e1 <= bar and e2 <= bar


# (f64, tiles, points, Gaussians, split): us split and on the tiles as measured
SPLIT = [
    (1, 508, 10, 0, False),   # 30.3, 15.6
    (1, 508, 0, 300, False),  # 336, 325
    (1, 128, 0, 300, True),   # 98, 172
    (1, 381, 63, 0, True),    # 40.5, 46.8
    (1, 576, 0, 300, True),   # 371, 433
    (0, 508, 10, 0, False),   # 15.2, 12.0
    (0, 477, 0, 30, False),   # 24.9, 20.4
    (0, 477, 40, 100, False),  # 63.1, 59.4
    (0, 128, 0, 30, True),    # 11.7, 15.0
    (0, 508, 0, 300, True),   # 125, 134
    (0, 672, 0, 300, False),
    (1, 128, 0, 0, False),
]


@pytest.mark.parametrize("case", SPLIT, ids=["-".join(map(str, c[:4])) for c in SPLIT])
def test_components_split_where_it_pays(rule, case):
    assert rule("split", *case[:4]) == case[4]


@pytest.mark.parametrize("f64,nt,n,uniform,small", [(1, 2, 1, 1, 0), (1, 2, 110, 1, 1), (1, 5, 110, 1, 0), (1, 5, 110, 0, 1),
                                                    (1, 16, 10, 0, 1), (0, 16, 10, 1, 0), (0, 40, 16, 1, 1), (0, 41, 16, 1, 0)])
def test_small_observations_split_where_it_pays(rule, f64, nt, n, uniform, small):
    assert rule("small", f64, nt, n, uniform) == small


# Few components on either side of the rules' lines: (tiles, times, channels, points, Gaussians)
FEW = [(16, 1, 8, 1, 0), (16, 1, 8, 15, 1), (45, 2, 16, 3, 2), (64, 2, 33, 16, 0), (100, 2, 25, 10, 0), (100, 2, 25, 0, 17),
       (128, 2, 47, 9, 65), (128, 3, 49, 1, 0), (128, 3, 49, 33, 31)]


@pytest.mark.gpu
@pytest.mark.parametrize("size", FEW, ids=["-".join(map(str, s)) for s in FEW])
@pytest.mark.parametrize("prec,dtype,bar", [(1, 0, 1e-6), (1, 1, 1e-6), (0, 0, 1e-11), (0, 1, 1e-6)])
def test_few_components_match_oracle(size, prec, dtype, bar):
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    from tests.test_pg_nodes import _case
    ctx = vp.vp_create_ctx(0, 0)
    try:
        for odd in (False, True):
            obs, sky = _case(*size, radius=0.2, odd=odd)
            ref = oracle.predict(obs, sky)
            # (noise below the few components' flux, so that the residual's own rounding to complex64 is below the bar)
            data = 0.1 * oracle.total_flux(obs, sky).min() * synth.noise_c64(ref.shape, 5).astype(np.complex128)
            data = data.astype(np.complex64).astype(np.complex128)
            with Handles(ctx, obs, sky) as h:
                got = run(ctx, h.obs, h.sky, obs, prec, dtype)
                res = run(ctx, h.obs, h.sky, obs, prec, dtype, data=data)
            e1, e2 = oracle.error_metric(got, ref, obs, sky), oracle.error_metric(res, data - ref, obs, sky)
            print(size, odd, "precision", prec, "dtype", dtype, "error / total flux %.2e %.2e" % (e1, e2), flush=True)
            assert e1 <= bar and e2 <= bar
    finally:
        vp.vp_destroy_ctx(ctx)
