"""Shapelets by nodes (csrc/shp_nodes.h): the number of Chebyshev nodes that the
library takes for an order and a band suffices for every Hermite function up to
that order along every line, on the CPU; on the GPU shapelets against the oracle on
channels around multiples of 16, with many shapelets, spectral terms, irregular
channels.  Observations as small as these go to the kernels by channels (csrc/dispatch.h):
test_shapelet_node_outputs.py has the sizes that the node kernels take."""
import dataclasses
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def node_count(tmp_path_factory):
    d = tmp_path_factory.mktemp("nodes")
    src = d / "n.cpp"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "%s"\n'
                   'int main(int c, char **v) { for (int i = 1; i + 2 < c; i += 3) '
                   'printf("%%d\\n", vp::shp_nodes(atoi(v[i]), 1.0, atof(v[i + 1]), atof(v[i + 2]))); }\n'
                   % os.path.join(ROOT, "paper_2005_09316_amd", "csrc", "shp_nodes.h"))
    exe = str(d / "n")
    subprocess.run(["g++", "-O1", "-std=c++17", str(src), "-o", exe], check=True)

    def run(args):
        out = subprocess.run([exe] + [repr(x) for a in args for x in a], check=True, capture_output=True, text=True)
        return [int(x) for x in out.stdout.split()]
    return run


def _hermite(nmax, x):
    p = np.zeros((nmax + 1,) + x.shape)
    p[0] = np.pi ** -0.25 * np.exp(-x * x / 2)
    if nmax:
        p[1] = np.sqrt(2) * x * p[0]
    for n in range(1, nmax):
        p[n + 1] = np.sqrt(2 / (n + 1)) * x * p[n] - np.sqrt(n / (n + 1)) * p[n - 1]
    return p


@pytest.mark.parametrize("tol", [1e-6, 1e-10, 1e-12])
def test_enough_nodes_for_every_line(node_count, tol):
    """Interpolation in nu on [1, hi] of phi_n(c nu), n <= N, over 60 lines c up
    to where the functions vanish: the error stays below twice the tolerance
    (the largest coefficient left out against their sum)."""
    cases = [(N, hi, tol) for N in (0, 1, 3, 10, 31, 54, 70, 96) for hi in (1.0014, 1.014, 1.06, 1.2, 1.4, 1.8)]
    for (N, hi, _), M in zip(cases, node_count(cases)):
        if M == 0:
            assert (N + 7) * (hi - 1) / 2 > 20  # refused only where very many would be needed
            continue
        h, mid = (hi - 1) / 2, (hi + 1) / 2
        k = np.arange(M)
        xn = np.cos(np.pi * (2 * k + 1) / (2 * M))
        w = (-1.0) ** k * np.sin(np.pi * (2 * k + 1) / (2 * M))
        x = np.linspace(-1, 1, 151) + 1e-9
        L = w / (x[:, None] - xn)
        L /= L.sum(1, keepdims=True)
        c = np.linspace(0, np.sqrt(2 * N + 2) + 6, 60)
        err = np.abs(_hermite(N, np.outer(c, mid + h * xn)) @ L.T - _hermite(N, np.outer(c, mid + h * x))).max()
        assert err <= 2 * tol + 1e-13, (N, hi, M, err)


CASES = {
    # (tiles, times, orders, frequencies)
    "narrow-16": (20, 2, [30, 7], synth.channels(182e6, 80e3, 16)),
    "narrow-17": (19, 3, [30], synth.channels(182e6, 80e3, 17)),
    "wide-96": (12, 2, [96, 0, 40], synth.band(150e6, 180e6, 96)),
    "wide-45": (9, 1, [54], synth.band(150e6, 180e6, 45)),
    "many-shapelets": (8, 2, [80, 11, 64, 63, 20, 33, 31, 32, 1, 70], synth.band(160e6, 180e6, 64)),
    "irregular": (17, 2, [47, 21], np.sort(np.random.default_rng(3).uniform(170e6, 190e6, 37))),
    # the middle channel is the middle of the band: a node where their number is odd
    "on-a-node": (10, 1, [22], synth.channels(182e6, 500e3, 33)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("prec,dtype,bar", [(0, 0, 1e-11), (1, 0, 1e-6), (1, 1, 1e-6), (0, 1, 1e-6)])
def test_nodes_match_oracle(name, prec, dtype, bar):
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    tiles, times, orders, freqs = CASES[name]
    obs, sky = synth.make_config(1, seed=77, n_tiles=tiles, n_time=times, n_chan=len(freqs), n_point=5, n_gauss=0,
                                 shapelet_nmax=orders, freq_hz=freqs)
    if name == "narrow-17":
        sky = synth.with_spectral_terms(sky, np.random.default_rng(4), 2)
    only = synth.select_components(sky, points=[], gauss=[])
    plus = dataclasses.replace(obs, sign=+1)
    data = synth.noise_c64((obs.n_time, obs.n_bl, obs.n_chan), 5).astype(np.complex128)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        for o, s, d in ((obs, sky, None), (plus, only, None), (obs, only, data)):
            ref = oracle.predict(o, s)
            with Handles(ctx, o, s) as h:
                got = run(ctx, h.obs, h.sky, o, prec, dtype, data=d)
            err = oracle.error_metric(got, ref if d is None else d - ref, o, s)
            print(name, "prec", prec, "dtype", dtype, "error / total flux %.2e" % err, flush=True)
            assert np.all(np.isfinite(got)) and err <= bar
    finally:
        vp.vp_destroy_ctx(ctx)


@pytest.mark.gpu
@pytest.mark.parametrize("n_point", [1, 4, 5])
@pytest.mark.parametrize("prec,dtype,bar", [(0, 0, 1e-11), (1, 0, 1e-6), (1, 1, 1e-6), (0, 1, 1e-6)])
def test_points_beside_nodes(n_point, prec, dtype, bar):
    """A few points go along with the shapelets' outputs (up to four), on
    regular and irregular channels, added to data and on their own."""
    import oracle
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, run
    ctx = vp.vp_create_ctx(0, 0)
    try:
        for name in ("narrow-17", "irregular"):
            tiles, times, orders, freqs = CASES[name]
            obs, sky = synth.make_config(1, seed=78, n_tiles=tiles, n_time=times, n_chan=len(freqs), n_point=n_point,
                                         n_gauss=0, shapelet_nmax=orders, freq_hz=freqs)
            ref = oracle.predict(obs, sky)
            data = synth.noise_c64(ref.shape, 5).astype(np.complex128)
            with Handles(ctx, obs, sky) as h:
                got = run(ctx, h.obs, h.sky, obs, prec, dtype)
                res = run(ctx, h.obs, h.sky, obs, prec, dtype, data=data)
            e1, e2 = oracle.error_metric(got, ref, obs, sky), oracle.error_metric(res, data - ref, obs, sky)
            print(name, n_point, "prec", prec, "dtype", dtype, "error / total flux %.2e %.2e" % (e1, e2), flush=True)
            assert e1 <= bar and e2 <= bar
    finally:
        vp.vp_destroy_ctx(ctx)
