"""Prefill and scoring passes of 257 to some thousand rows: where the projections change kernels (rotary and SwiGLU in the
epilogue or behind it, 128 x 128 or 256 x 256 tiles, K splits), at widths on either side of those points."""
from dataclasses import replace

import numpy as np
import pytest

from tests import stage_harness as H
from workload import CONFIGS

pytestmark = pytest.mark.gpu

_GPT2S = CONFIGS["gpt2s"]
_NARROW = replace(_GPT2S.model, n_layers=2, d_model=320, n_q_heads=5, n_kv_heads=5, head_dim=64, ffn=448, vocab=1003)
_MIDDLE = replace(_NARROW, d_model=1088, n_q_heads=17, n_kv_heads=17, ffn=1600)
# few tiles of QKV, more than half a round of gate||up
_SKEWED = replace(_NARROW, n_layers=1, d_model=1600, n_q_heads=8, n_kv_heads=1, head_dim=128, ffn=16640)

# 2300 rows: O adds to the residual stream, with 64 columns and some 250 rows in the last tiles
_ADDING = replace(_NARROW, n_layers=1, d_model=2112, n_q_heads=16, n_kv_heads=2, head_dim=128, ffn=1088)


@pytest.mark.parametrize("model,n,prompt", [(_NARROW, 2, 128), (_NARROW, 3, 170), (_MIDDLE, 2, 130), (_MIDDLE, 3, 149),
                                            (_MIDDLE, 5, 140), (_SKEWED, 2, 140), (_ADDING, 16, 142)])
def test_passes_beyond_256_rows(model, n, prompt):
    cfg = _GPT2S.with_(name="mid_passes", model=model, n_samples=n, prompt_len=(prompt, prompt + 2), gain_jitter=0.05)
    ref = H.oracle_stage(cfg, n=n, max_len=3, dtype=np.float32)
    got = H.run_gpu_stage(cfg, ref, fused=False, R_t=0, chunk_tokens=1 << 20, max_batch_tokens=4096)
    H.compare_stage(cfg, ref, got)
    half = H.run_gpu_stage(cfg, ref, fused=False, R_t=0, chunk_tokens=1 << 20, max_batch_tokens=4096, half_weight_copies=True)
    for k in ("tokens", "lp_actor", "lp_ref", "values", "reward", "lp_actor_rescored"):
        np.testing.assert_array_equal(got[k], half[k], err_msg=k)
