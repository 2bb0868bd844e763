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
