"""Threads that launch the same kernels with different amounts of LDS (other orders,
node counts, tiles), each on a stream of its own: every result is that of a call
alone, and no launch is refused."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _pairs():
    out = []
    for i, (tiles, chans, points, radius, orders) in enumerate(((30, 64, 300, 0.002, [8]), (64, 40, 900, 0.008, [60]),
                                                                (128, 26, 1500, 0.2, [30, 20, 12, 9, 8, 31]),
                                                                (129, 64, 321, 0.2, [5]))):
        obs, sky = synth.make_config(1, seed=50 + i, n_tiles=tiles, n_time=4, n_chan=chans, n_point=points, n_gauss=20,
                                     shapelet_nmax=orders, freq_hz=synth.channels(182e6, 80e3, chans))
        rng = np.random.default_rng(i)
        for n, ra, dec in ((points, "p_ra", "p_dec"), (20, "g_ra", "g_dec")):
            r, th = radius * np.sqrt(rng.random(n)), 2 * np.pi * rng.random(n)
            setattr(sky, dec, obs.dec0 + r * np.sin(th))
            setattr(sky, ra, obs.ra0 + r * np.cos(th) / np.cos(obs.dec0))
        out.append((obs, sky))
    return out


def test_predict_from_threads():
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    ctx = vp.vp_create_ctx(0, 0)
    try:
        pairs = _pairs()
        hs = [Handles(ctx, *p) for p in pairs]
        shape = [(o.n_time, o.n_bl, o.n_chan) for o, _ in pairs]
        precs = (vp.VP_PREC_MIXED, vp.VP_PREC_FP64)

        def call(i, prec, t, stream):
            vp.vp_predict(ctx, hs[i].sky, hs[i].obs, prec, vp.VP_C128, t.data_ptr(), stream.cuda_stream)
        main = torch.cuda.current_stream()
        want = {}
        for i in range(4):
            for p in precs:
                want[i, p] = torch.empty(shape[i], dtype=torch.complex128, device="cuda")
                call(i, p, want[i, p], main)
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in range(4)]
        got = [[torch.empty(shape[i], dtype=torch.complex128, device="cuda") for _ in range(6)] for i in range(4)]
        torch.cuda.synchronize()
        errors = []

        def work(i):
            try:
                for r in range(6):
                    call(i, precs[r % 2], got[i][r], streams[i])
            except Exception as e:  # noqa: BLE001  (any refusal fails the test)
                errors.append((i, e))
        threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert not errors
        for i in range(4):
            for r in range(6):
                assert torch.equal(torch.view_as_real(got[i][r]), torch.view_as_real(want[i, precs[r % 2]])), (i, r)
        for h in hs:
            h.close()
    finally:
        vp.vp_destroy_ctx(ctx)


def test_peels_from_contexts_of_their_own():
    """Two contexts, two threads, solves of 30 and of 100 tiles (one kernel each for up
    to 64 and 128, and the same one for 100 and 128)."""
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    ctxs, work_on = [], []
    try:
        for n in (100, 128):
            ctx = vp.vp_create_ctx(0, 0)
            ctxs.append(ctx)
            obs, sky = synth.make_config(1, seed=n, n_tiles=n, n_time=1, n_chan=8, n_point=1, n_gauss=0, shapelet_nmax=[12])
            h = Handles(ctx, obs, sky)
            data = torch.empty((obs.n_time, obs.n_bl, obs.n_chan), dtype=torch.complex128, device="cuda")
            vp.vp_predict(ctx, h.sky, h.obs, vp.VP_PREC_FP64, vp.VP_C128, data.data_ptr(), 0)
            torch.cuda.synchronize()
            work_on.append((ctx, h, n, synth.antenna_pairs(n), 1.21 * data))
        streams, errors = [torch.cuda.Stream() for _ in range(2)], []
        left = [[w[4].clone() for _ in range(4)] for w in work_on]
        torch.cuda.synchronize()

        def work(i):
            ctx, h, n, (a1, a2), _ = work_on[i]
            try:
                for r in range(4):
                    vp.vp_peel(ctx, h.sky, h.obs, a1, a2, n, 12, (vp.VP_PREC_FP64, vp.VP_PREC_MIXED)[r % 2], vp.VP_C128,
                               left[i][r].data_ptr(), 0, streams[i].cuda_stream)
            except Exception as e:  # noqa: BLE001
                errors.append((i, e))
        threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert not errors
        for i in range(2):
            top = float(work_on[i][4].abs().max())
            for r in range(4):
                assert float(left[i][r].abs().max()) <= (1e-9 if r % 2 == 0 else 1e-5) * top
            work_on[i][1].close()
    finally:
        for ctx in ctxs:
            vp.vp_destroy_ctx(ctx)
