"""vp_serve_stats: the time with a job on the device is the union of the jobs' device
intervals, however often and whenever it is asked for, and the kernels counted are
those that the jobs launched."""
import os
import subprocess
import time

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("seed,jobs", [(1, 200), (2, 2000), (3, 20000)])
def test_union_of_intervals(tmp_path, seed, jobs):
    exe = str(tmp_path / "spans")
    subprocess.run(["g++", "-O1", "-std=c++17", os.path.join(ROOT, "tests", "serve_spans_test.cpp"), "-o", exe], check=True)
    wrong, held = map(int, subprocess.run([exe, str(seed), str(jobs)], check=True, capture_output=True,
                                          text=True).stdout.split())
    assert wrong == 0
    assert held <= 2 * 4096


@pytest.mark.gpu
def test_stats_of_a_stream():
    """Asked after every completion: the time never exceeds the span of the jobs'
    device clocks, ends at their union, and every job's passes are counted, with the
    tables of the pairs (two kernels, two more where points may go by antenna)."""
    import torch
    from paper_2005_09316_amd import vp
    from tests.helpers import Handles, vis_tensor
    ctx = vp.vp_create_ctx(0, 0)
    try:
        specs = [synth.make_config(1, seed=20 + i, n_tiles=32 + 8 * i, n_time=2, n_chan=24, n_point=40 * (i + 1), n_gauss=9,
                                   shapelet_nmax=[20]) for i in range(3)]
        # the first job outlasts the others, which end while it runs
        long = synth.make_config(1, seed=30, n_tiles=128, n_time=14, n_chan=64, n_point=20000, n_gauss=3000, shapelet_nmax=[20])
        hs = [Handles(ctx, o, s) for o, s in specs] + [Handles(ctx, *long)]
        which = [3] + [i % 3 for i in range(24)]
        bufs = [vis_tensor((specs + [long])[k][0], vp.VP_C64) for k in which]
        torch.cuda.synchronize()
        tickets = [vp.vp_submit(ctx, vp.VP_JOB_PREDICT, hs[k].sky, hs[k].obs, vp.VP_PREC_MIXED, vp.VP_C64, b.data_ptr())
                   for k, b in zip(which, bufs)]
        done, last, t0 = {}, 0.0, time.time()
        while len(done) < len(tickets) and time.time() - t0 < 60:
            for t in tickets:
                if t not in done:
                    r = vp.vp_poll(ctx, t)
                    if r is not None:
                        assert r["status"] == vp.VP_OK
                        done[t] = r
                        ms = vp.vp_serve_stats(ctx)[1]
                        assert ms >= last
                        last = ms
        assert len(done) == len(which)
        launches, ms = vp.vp_serve_stats(ctx)
        iv = sorted((r["dev_first_tile"], r["dev_last_tile"]) for r in done.values())
        covered, end = 0, 0
        for a, b in iv:
            covered += max(0, b - max(a, end))
            end = max(end, b)
        # one clock rate for all: ticks per ms from the union itself, a round number of kHz
        rate = covered / ms
        assert abs(rate / 100000.0 - 1.0) < 1e-9, rate
        # per job a point/Gaussian and a shapelet pass at least, three where by antenna
        assert 2 * len(which) + 2 * 4 <= launches <= 3 * len(which) + 4 * 4
        for h in hs:
            h.close()
    finally:
        vp.vp_destroy_ctx(ctx)
