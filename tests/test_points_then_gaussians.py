"""Points by antenna beside Gaussians, into complex64 on the mixed path: the two
passes' sums meet in FP64 and are rounded once.  The same call into complex128
keeps them in FP64 throughout, so its result rounded to complex64 is the
complex64 call's, bit for bit; subtracting adds the data's own FP64 rounding.
Sizes: one part, several parts by time steps and by channels, Gaussians by
channels and by nodes."""
import dataclasses

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CASES = {
    # name: (tiles, times, channels, points, Gaussians, field radius rad, noalloc too)
    "wide": (64, 6, 33, 1500, 20, 0.2, True),
    "irregular": (40, 14, 36, 1471, 7, 0.2, True),
    "odd-channels": (96, 4, 35, 703, 3, 0.2, True),
    "by-nodes": (128, 2, 96, 1500, 65, 0.003, True),
    "times-in-parts": (128, 14, 160, 300, 5, 0.2, False),
    "noalloc-times-in-parts": (128, 6, 130, 320, 5, 0.2, True),
    "noalloc-channels-in-parts": (256, 1, 163, 320, 5, 0.2, True),
    "noalloc-channels-in-parts-by-nodes": (256, 1, 200, 2000, 40, 0.012, True),
}


def _inputs(name):
    tiles, times, chans, points, gauss, radius, _ = CASES[name]
    freqs = synth.channels(182e6, 80e3, chans)
    if name == "irregular":
        freqs = np.sort(np.random.default_rng(8).uniform(175e6, 185e6, chans))
    obs, sky = synth.make_config(1, seed=70 + tiles, n_tiles=tiles, n_time=times, n_chan=chans, n_point=points,
                                 n_gauss=gauss, shapelet_nmax=[], freq_hz=freqs)
    rng = np.random.default_rng(tiles)
    for n, ra, dec in ((points, "p_ra", "p_dec"), (gauss, "g_ra", "g_dec")):
        r, th = radius * np.sqrt(rng.random(n)), 2 * np.pi * rng.random(n)
        setattr(sky, dec, obs.dec0 + r * np.sin(th))
        setattr(sky, ra, obs.ra0 + r * np.cos(th) / np.cos(obs.dec0))
    return dataclasses.replace(obs, beam_fwhm_rad=0.0), sky


def _call(fn, ctx, h, t, stream):
    from paper_2005_09316_amd import vp
    dtype = vp.VP_C64 if t.is_complex() and t.element_size() == 8 else vp.VP_C128
    fn(ctx, h.sky, h.obs, vp.VP_PREC_MIXED, dtype, t.data_ptr(), stream.cuda_stream)


@pytest.mark.parametrize("name", sorted(CASES))
def test_rounded_once(name):
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    obs, sky = _inputs(name)
    shape = (obs.n_time, obs.n_bl, obs.n_chan)
    stream = torch.cuda.current_stream()
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            wide = torch.empty(shape, dtype=torch.complex128, device="cuda")
            got = torch.empty(shape, dtype=torch.complex64, device="cuda")
            vp.vp_profile(ctx, True)
            _call(vp.vp_predict, ctx, h, wide, stream)
            counts, _ = vp.vp_profile_read(ctx)
            assert counts[1] == 2, counts  # by antenna, then the Gaussians
            _call(vp.vp_predict, ctx, h, got, stream)
            counts, _ = vp.vp_profile_read(ctx)
            assert counts[1] == (4 if name == "times-in-parts" else 2), counts
            assert torch.equal(torch.view_as_real(got), torch.view_as_real(wide.to(torch.complex64)))
            if CASES[name][-1]:
                other = torch.empty_like(got)
                _call(vp.vp_predict_noalloc, ctx, h, other, stream)
                stream.synchronize()
                assert torch.equal(torch.view_as_real(got), torch.view_as_real(other))
            # the residual: the data's complex64 values less the FP64 sum, rounded once
            data = wide.to(torch.complex64) * (1 + 2.0 ** -10)
            res64, res = data.to(torch.complex128), data.clone()
            _call(vp.vp_subtract, ctx, h, res64, stream)
            _call(vp.vp_subtract, ctx, h, res, stream)
            stream.synchronize()
            a, b = torch.view_as_real(res).double(), torch.view_as_real(res64)
            big = torch.view_as_real(data).abs().double()
            # half an ulp of the residual, and the data's FP64 rounding in either call
            off = (a - b).abs() - (2.0 ** -24 * b.abs() + 2.0 ** -51 * big + 1e-40)
            assert float(off.max()) <= 0.0
    finally:
        vp.vp_destroy_ctx(ctx)


def test_on_several_streams_and_threads():
    """Six streams from three threads share the context's workspaces: every
    result is the one of a call alone."""
    import threading
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    obs, sky = _inputs("wide")
    shape = (obs.n_time, obs.n_bl, obs.n_chan)
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            ref = torch.empty(shape, dtype=torch.complex64, device="cuda")
            _call(vp.vp_predict, ctx, h, ref, torch.cuda.current_stream())
            torch.cuda.synchronize()
            streams = [torch.cuda.Stream() for _ in range(6)]
            outs = [torch.empty((8,) + shape, dtype=torch.complex64, device="cuda") for _ in streams]
            torch.cuda.synchronize()

            def work(i):
                for r in range(8):
                    for s in (2 * i, 2 * i + 1):
                        _call(vp.vp_predict, ctx, h, outs[s][r], streams[s])
            threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
            for t in threads:
                t.start()
            for t in threads:
                t.join()
            torch.cuda.synchronize()
            want = torch.view_as_real(ref)
            assert all(torch.equal(torch.view_as_real(o[r]), want) for o in outs for r in range(8))
    finally:
        vp.vp_destroy_ctx(ctx)
