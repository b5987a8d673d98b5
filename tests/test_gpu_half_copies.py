"""Decode steps with and without half copies of the weights, at widths where the copies are read and row counts
around the points where kernels change: bit-identical, whatever the widths do to K splits and shares of K."""
from dataclasses import replace

import numpy as np
import pytest

from tests import stage_harness as H
from workload import CONFIGS

pytestmark = pytest.mark.gpu

_GPT2S = CONFIGS["gpt2s"]
_BASE = replace(_GPT2S.model, n_layers=1, d_model=4096, n_q_heads=32, n_kv_heads=4, head_dim=128, ffn=704, vocab=4100)
# K of 17 steps of 64, fewer weight rows than one block a compute unit
_NARROW = replace(_BASE, d_model=1088, n_q_heads=8, n_kv_heads=1, ffn=1600)
# another number of planes behind O and down
_ODD = replace(_BASE, d_model=5120, n_q_heads=40, n_kv_heads=5, ffn=2112)
_WIDEST = replace(_BASE, d_model=8192, n_q_heads=16, n_kv_heads=2, vocab=1030)


@pytest.mark.parametrize("model,n", [(_BASE, 32), (_BASE, 33), (_BASE, 64), (_BASE, 65), (_NARROW, 40), (_ODD, 50), (_WIDEST, 36), (_WIDEST, 70)])
def test_half_copies_do_not_change_decode_results(model, n):
    cfg = _GPT2S.with_(name="half_copies", model=model, n_samples=n, prompt_len=(3, 5), gain_jitter=0.05)
    inp = H.make_inputs(cfg, n=n, max_len=4, weight_device="cuda")
    a, b = (H.run_gpu_stage(cfg, inp, fused=False, R_t=0, chunk_tokens=64, half_weight_copies=half) for half in (False, True))
    for k in ("tokens", "lp_actor", "lp_ref", "values", "reward", "lp_actor_rescored"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
