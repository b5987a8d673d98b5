"""Batch passes of 3072 rows and more without half copies convert each matrix into a workspace first: the same bits as
with half copies made once, and as the conversion itself element by element."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import paper_2409_13221_amd as R
from tests import stage_harness as H
from workload import CONFIGS

pytestmark = pytest.mark.gpu

_GPT2S = CONFIGS["gpt2s"]
# every projection on the tall kernel, with ragged last tiles; and widths where O and down stay on 128 x 128 tiles
_WIDE = replace(_GPT2S.model, n_layers=2, d_model=1088, n_q_heads=17, n_kv_heads=17, head_dim=64, ffn=1152, vocab=515)
_NARROW = replace(_WIDE, d_model=256, n_q_heads=4, n_kv_heads=4, ffn=704)


@pytest.mark.parametrize("model,n,prompt", [(_WIDE, 3, 1023), (_WIDE, 3, 1024), (_WIDE, 8, 517), (_NARROW, 8, 517)])
def test_converted_weights_do_not_change_results(model, n, prompt):
    cfg = _GPT2S.with_(name="converted", model=model, n_samples=n, prompt_len=(prompt, prompt), gain_jitter=0.05)
    inp = H.make_inputs(cfg, n=n, max_len=2, weight_device="cuda")
    a, b = (H.run_gpu_stage(cfg, inp, fused=False, R_t=0, chunk_tokens=8192, half_weight_copies=half, max_batch_tokens=8192)
            for half in (False, True))
    for k in ("tokens", "lp_actor", "lp_ref", "values", "reward", "lp_actor_rescored"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


def test_conversions_hold_no_memory_of_their_own():
    def taken(half):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        ctx = R.rlhf_create(R.rlhf_model_cfg(1, 4096, 32, 32, 128, 11008, 515, R.RLHF_BF16, 1e-5, 10000.0),
                            R.rlhf_engine_cfg(16, 1 << 24, 4, 64, 4, 3072, 2, 0, 0, 0, None, None, half))
        used = before - torch.cuda.mem_get_info()[0]
        R.rlhf_destroy(ctx)
        return used
    taken(1)
    assert abs(taken(0) - taken(1)) <= 16 << 20            # a converted gate || up matrix would be 180 MB


def test_profiled_projections_include_their_conversion():
    """A pass of 3072 rows over one wide layer: about 0.8 GB of conversions beside 1.2 ms of projections on half weights."""
    cfg = _GPT2S.with_(name="converted_profile", n_samples=6, prompt_len=(512, 512),
                       model=replace(_GPT2S.model, n_layers=1, d_model=4096, n_q_heads=32, n_kv_heads=32, head_dim=128, ffn=11008, vocab=515))
    inp = H.make_inputs(cfg, n=6, max_len=1, weight_device="cuda")
    ms = []
    for half in (False, True):
        with H.GpuStage(cfg, inp, max_batch_tokens=3072, half_weight_copies=half) as st:
            best = []
            for _ in range(8):
                st.submit()
                R.rlhf_profile_begin(st.ctx, 1)
                R.rlhf_generate_step(st.ctx)
                p = R.rlhf_profile_end(st.ctx)["gemm_batch"]
                assert p["sampled"] == p["launches"] and p["dropped"] == 0
                best.append(p["sampled_ms"])
            ms.append(min(best[2:]))
    print("projections, ms, converted and with copies:", ms)
    assert ms[0] > ms[1] + 0.06                            # at 8 TB/s they take 0.1 ms


@pytest.mark.parametrize("n", [2, 6, 8, 14, 4096, 4096 * 1024 + 6])
@pytest.mark.parametrize("offset", [0, 2, 8])
def test_conversion_at_any_length_and_alignment(n, offset):
    src = (torch.randn(n + offset, device="cuda") * 3).to(torch.bfloat16)[offset:]
    want = src.float().clamp(-65504, 65504).half()         # these values are exact in half but for subnormal ones
    got = R.rlhf_op_bf16_to_half(src)
    assert float((got.float() - want.float()).abs().max()) <= 2.0 ** -24
