"""fused = 2 on both sides of one scoring pass of tokens, and the same results under either plan."""
import numpy as np
import pytest

from tests import stage_harness as H
from workload import CONFIGS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,fused", [(100, 0), (260, 1)])
def test_small_models_run_fused_beyond_one_scoring_pass(n, fused):
    cfg = CONFIGS["tiny"].with_(name="plan_choice", n_samples=n, gain_jitter=0.05)
    inp = H.make_inputs(cfg, n=n, max_len=16)
    tokens = int(np.diff(inp["prompt_offsets"]).sum() + inp["out_len"].sum())
    assert (tokens >= 10000) == bool(fused)
    res = []
    for plan in ("auto", 1 - fused):
        with H.GpuStage(cfg, inp) as g:
            g.submit(None)
            stats, _ = g.R.rlhf_run_stage(g.ctx, plan if plan == "auto" else bool(plan), n + 1, 2048, H.ALL_ROLES)
            assert stats.fused_used == (fused if plan == "auto" else 1 - fused)
            res.append(g.results())
    np.testing.assert_array_equal(res[0]["tokens"], res[1]["tokens"])
    for k in ("lp_actor", "lp_ref", "values"):
        np.testing.assert_allclose(res[0][k], res[1][k], rtol=0, atol=1e-4)
