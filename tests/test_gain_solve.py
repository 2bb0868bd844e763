"""The gain solve with both tables of a cell on chip (csrc/vp_calib.hip,
k_gain_pairs and k_gain_solve_rw) at its edges: 64 and 128 tiles, one to each
side, every tile with baselines, some of them flagged and some with the tiles in
the other order, cells that do not fill a table workgroup.  Against
oracle.peel, with the peel's own bars (tests/test_peel_gpu.py)."""
import numpy as np
import pytest

import oracle
import synth
from paper_2005_09316_amd import vp
from tests.test_peel_gpu import GAIN_FACTOR, PRED_BAR, RES_FACTOR, _input_as, _make, _res_err, _run_peel, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,dtype", [(vp.VP_PREC_FP64, vp.VP_C128), (vp.VP_PREC_FP64, vp.VP_C64),
                                        (vp.VP_PREC_MIXED, vp.VP_C64), (vp.VP_PREC_MIXED, vp.VP_C128)])
@pytest.mark.parametrize("n", [2, 31, 63, 64, 65, 127, 128, 129])
def test_gain_solve_edges(ctx, n, prec, dtype):  # noqa: F811
    rng = np.random.default_rng(100 + n)
    nb = n * (n - 1) // 2
    keep = np.sort(rng.choice(nb, max(1, int(0.8 * nb)), replace=False))
    if n > 2:  # the baselines of tile 0 stay, so that the graph is connected
        keep = np.union1d(keep, np.flatnonzero(synth.antenna_pairs(n)[0] == 0))
    swap = rng.random(keep.size) < 0.3
    obs, sky, a1, a2, n_ant, data, M = _make(n_tiles=n, n_time=1, n_chan=3, keep=keep, swap=swap, seed=n)
    data = _input_as(data, dtype)
    g, res = _run_peel(ctx, obs, sky, a1, a2, n_ant, data, 6, prec, dtype)
    g_ref, res_ref = oracle.peel(data, M, a1, a2, n_ant, 6)
    p, p_ref = g[:, :, a1] * np.conj(g[:, :, a2]), g_ref[:, :, a1] * np.conj(g_ref[:, :, a2])
    ep = np.abs(p - p_ref).max() / np.abs(p_ref).max()
    er = _res_err(res, res_ref, obs, sky)
    bar = max(PRED_BAR[prec], 1e-6 if dtype == vp.VP_C64 else 0.0)
    print("gain solve n", n, "precision", prec, "dtype", dtype, "g_i g_j^* %.2e, residual / F %.2e" % (ep, er), flush=True)
    assert np.all(np.isfinite(g)) and np.all(np.isfinite(res))
    assert ep <= GAIN_FACTOR * bar and er <= RES_FACTOR * bar
