"""A point far brighter than the others, wherever it stands in the list: the mixed
path's FP32 groups add it last, so that its visibilities are hardly less exact than
on its own."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("at", [0, 3, 7])
@pytest.mark.parametrize("n_time", [1, 14])
def test_faint_points_cost_a_bright_one_one_rounding(at, n_time):
    """Seven points of 1e-4 Jy beside one of 1 Jy.  Alone its FP32 sine, cosine and
    product leave e0, some 1.3e-7 rms as a complex number; each further addition at its
    size rounds both parts by at most 1.7e-8 rms (a uniform half ulp of 2^-24).  One of
    them and the pair's: e1 <= sqrt(e0^2 + 4 x 1.7e-8^2) = 1.04 e0 at most; with the
    seven behind it, 1.09 was measured."""
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    rng = np.random.default_rng(11)
    obs = synth.make_obs(rng, 128, n_time, synth.channels(182e6, 80e3, 32))
    sky = synth.make_sky(rng, n_point=8, n_gauss=0, shapelet_nmax=[], cap_rad=math.radians(9.0),
                         point_flux=synth._pl(0.05, 50.0), shapelet_sref=synth._lu(20.0, 200.0), tau=20.0)
    sky.p_alpha = np.zeros(8)
    sky.p_sref = np.where(np.arange(8) == at, 1.0, 1e-4)
    one = synth.select_components(sky, points=[at])
    ctx = vp.vp_create_ctx(0, 0)
    rms = []
    try:
        for s in (one, sky):
            with Handles(ctx, obs, s) as h:
                a = torch.empty((obs.n_time, obs.n_bl, obs.n_chan), dtype=torch.complex128, device="cuda")
                b = torch.empty_like(a)
                vp.vp_predict(ctx, h.sky, h.obs, vp.VP_PREC_FP64, vp.VP_C128, a.data_ptr(), 0)
                vp.vp_predict(ctx, h.sky, h.obs, vp.VP_PREC_MIXED, vp.VP_C128, b.data_ptr(), 0)
                torch.cuda.synchronize()
                rms.append(float((a - b).abs().square().mean().sqrt()))
    finally:
        vp.vp_destroy_ctx(ctx)
    print("rms error alone %.3e, with seven faint ones %.3e" % tuple(rms), flush=True)
    assert rms[1] <= 1.05 * rms[0]
