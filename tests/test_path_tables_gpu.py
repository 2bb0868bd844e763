"""Per-(sky, observation) tables: the components' own are built by a pair's first call,
what a precision path's kernels by nodes and by antenna need beside them by the first
call on that path.  Results do not depend on the order of calls, streams or threads,
and a call under capture whose path's tables are not there does without them."""
import itertools

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _inputs():
    """Points by antenna, Gaussians by nodes, shapelets by nodes, on both paths."""
    rng = np.random.default_rng(5)
    obs, sky = synth.make_config(1, seed=9, n_tiles=128, n_time=4, n_chan=96, n_point=1500, n_gauss=40, shapelet_nmax=[20],
                                 freq_hz=synth.channels(182e6, 80e3, 96))
    for n, ra, dec in ((1500, "p_ra", "p_dec"), (40, "g_ra", "g_dec")):
        r, th = 0.01 * np.sqrt(rng.random(n)), 2 * np.pi * rng.random(n)
        setattr(sky, dec, obs.dec0 + r * np.sin(th))
        setattr(sky, ra, obs.ra0 + r * np.cos(th) / np.cos(obs.dec0))
    return obs, sky


def _run(ctx, h, obs, prec, stream=None):
    import torch
    from paper_2005_09316_amd import vp
    t = torch.empty((obs.n_time, obs.n_bl, obs.n_chan), dtype=torch.complex128, device="cuda")
    s = stream or torch.cuda.current_stream()
    s.wait_stream(torch.cuda.current_stream())
    vp.vp_predict(ctx, h.sky, h.obs, prec, vp.VP_C128, t.data_ptr(), s.cuda_stream)
    return t


def test_every_order_gives_the_same():
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    obs, sky = _inputs()
    precs = (vp.VP_PREC_MIXED, vp.VP_PREC_FP64, vp.VP_PREC_FP32)
    alone = {}
    for p in precs:
        ctx = vp.vp_create_ctx(0, 0)
        with Handles(ctx, obs, sky) as h:
            alone[p] = _run(ctx, h, obs, p)
            torch.cuda.synchronize()
        vp.vp_destroy_ctx(ctx)
    streams = [torch.cuda.Stream() for _ in range(3)]
    for order in itertools.permutations(precs):
        ctx = vp.vp_create_ctx(0, 0)
        try:
            with Handles(ctx, obs, sky) as h:
                vp.vp_profile(ctx, True)
                # each path's first call at once, on a stream of its own
                got = [(p, _run(ctx, h, obs, p, streams[i])) for i, p in enumerate(order)]
                got += [(p, _run(ctx, h, obs, p, streams[(i + 1) % 3])) for i, p in enumerate(order)]
                torch.cuda.synchronize()
                counts, _ = vp.vp_profile_read(ctx)
                # builds: with the first call, and by each further path's first (FP32 has none of its own)
                first_has_none = order[0] == vp.VP_PREC_FP32
                assert counts[0] == (3 if first_has_none else 2), (order, counts)
                for p, t in got:
                    assert torch.equal(torch.view_as_real(t), torch.view_as_real(alone[p])), (order, p)
        finally:
            vp.vp_destroy_ctx(ctx)


def test_threads_share_the_first_build():
    import threading
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    obs, sky = _inputs()
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            streams = [torch.cuda.Stream() for _ in range(6)]
            outs = [torch.empty((obs.n_time, obs.n_bl, obs.n_chan), dtype=torch.complex128, device="cuda") for _ in streams]
            torch.cuda.synchronize()
            gate = threading.Barrier(6)

            def work(i):
                gate.wait()
                vp.vp_predict(ctx, h.sky, h.obs, (vp.VP_PREC_MIXED, vp.VP_PREC_FP64)[i % 2], vp.VP_C128,
                              outs[i].data_ptr(), streams[i].cuda_stream)
            threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
            for t in threads:
                t.start()
            for t in threads:
                t.join()
            torch.cuda.synchronize()
            for i in range(2, 6):
                assert torch.equal(torch.view_as_real(outs[i]), torch.view_as_real(outs[i % 2]))
            d = (outs[0] - outs[1]).abs().max() / outs[1].abs().max()
            assert 0 < float(d) < 1e-6
    finally:
        vp.vp_destroy_ctx(ctx)


def test_capture_without_the_paths_tables():
    """FP64 captured after a mixed call only, then eager FP64 (which builds its tables),
    with replays between: all within the path's bar of each other, replays bitwise alike."""
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles
    obs, sky = _inputs()
    ctx = vp.vp_create_ctx(0, 0)
    try:
        with Handles(ctx, obs, sky) as h:
            _run(ctx, h, obs, vp.VP_PREC_MIXED)
            out = torch.zeros((obs.n_time, obs.n_bl, obs.n_chan), dtype=torch.complex128, device="cuda")
            torch.cuda.synchronize()
            s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                vp.vp_predict(ctx, h.sky, h.obs, vp.VP_PREC_FP64, vp.VP_C128, out.data_ptr(), s.cuda_stream)
            seen = []
            for i in range(3):
                out.zero_()
                g.replay()
                torch.cuda.synchronize()
                seen.append(out.clone())
                eager = _run(ctx, h, obs, vp.VP_PREC_FP64)
                torch.cuda.synchronize()
                err = float((out - eager).abs().max()) / float(eager.abs().max())
                print("replay", i, "against eager %.2e" % err, flush=True)
                assert err <= 1e-11
            assert all(torch.equal(torch.view_as_real(x), torch.view_as_real(seen[0])) for x in seen)
            # captured again, with the tables: the eager call's own kernels
            g2 = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g2, stream=s):
                vp.vp_predict(ctx, h.sky, h.obs, vp.VP_PREC_FP64, vp.VP_C128, out.data_ptr(), s.cuda_stream)
            for i in range(3):
                out.zero_()
                g2.replay()
                torch.cuda.synchronize()
                assert torch.equal(torch.view_as_real(out), torch.view_as_real(eager))
            del g, g2
    finally:
        vp.vp_destroy_ctx(ctx)
