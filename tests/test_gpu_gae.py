"""Advantages, returns and packed results at the edges of their kernels' tiles: lengths around 8, 64, 512
and 2048 tokens, and enough tokens that the results leave in more than one piece."""
from dataclasses import replace

import numpy as np
import pytest

from oracle.gae import gae, token_rewards
from tests import stage_harness as H
from workload import CONFIGS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gamma,lam", [(0.99, 0.95), (1.0, 1.0), (0.9, 0.0)])
def test_gae_and_packed_results_at_tile_edges(gamma, lam):
    lens = np.array([1, 7, 8, 9, 63, 64, 65, 511, 512, 513, 2047, 2048, 2049] + [2300] * 88, np.int32)
    tiny = CONFIGS["tiny"]
    cfg = tiny.with_(name="gae_edges", model=replace(tiny.model, n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, ffn=64, vocab=128), n_samples=len(lens),
                     prompt_len=(1, 3))
    inp = H.make_inputs(cfg, n=len(lens))
    inp["out_len"] = lens
    with H.GpuStage(cfg, inp) as g:
        g.submit()
        g.R.rlhf_run_stage(g.ctx, False, 0, 8192, 0b1111)
        res = g.results()
        adv, ret = g.R.rlhf_compute_gae(g.ctx, gamma, lam, 0.1, int(lens.sum()))
    o = res["resp_offsets"]
    assert np.diff(o).tolist() == lens.tolist() and o[-1] * 5 > 1 << 20
    # decoding and the re-scoring forward see the same tokens: packed rows are where they belong
    np.testing.assert_allclose(res["lp_actor"], res["lp_actor_rescored"], rtol=0, atol=1e-4)
    assert (res["tokens"][o[1:] - 1] == cfg.eos_id).all()
    for i, L in enumerate(lens):
        s = slice(o[i], o[i + 1])
        a, r = gae(token_rewards(res["lp_actor"][s], res["lp_ref"][s], res["reward"][i], 0.1), res["values"][s], gamma, lam)
        # float32 sums of up to L terms (gamma = lam = 1) against float64: roundoff 6e-8 a step, on partial
        # sums no larger than the sum of the terms' sizes
        tol = 6e-8 * (12 if gamma * lam < 1 else 12 + L / 16) * (np.abs(a).max() + np.abs(r).max() + 1.0)
        np.testing.assert_allclose(adv[s], a, rtol=0, atol=tol)
        np.testing.assert_allclose(ret[s], r, rtol=0, atol=tol)
