"""Decode steps (and short prefills) of 1..256 rows run on the weight-streaming projections: batch sizes
at the edges of their row blocks, a model whose sizes leave remainders in every projection, and one
wide enough for several weight blocks per workgroup and for K splits.  The oracle generates; log-probs,
values and rewards are held to the tolerances of the other stage tests."""
from dataclasses import replace

import numpy as np
import pytest

from tests import stage_harness as H
from workload import CONFIGS, make_weights, make_workload

pytestmark = pytest.mark.gpu

_GPT2S = CONFIGS["gpt2s"]
# 5 steps of 64 along d and 7 along ffn: waves with no step of their own; a ragged vocabulary
_SMALL = replace(_GPT2S.model, n_layers=2, d_model=320, n_q_heads=5, n_kv_heads=5, head_dim=64, ffn=448, vocab=1003)
# N >= 4096 everywhere but in the KV heads' share, K = 4096 and 704
_WIDE = replace(_GPT2S.model, n_layers=1, d_model=4096, n_q_heads=32, n_kv_heads=4, head_dim=128, ffn=704, vocab=4100)
# the float model's own kernel: K with half a chunk of 16 left over, a ragged vocabulary
_FLOAT = replace(_SMALL, d_model=208, n_q_heads=2, n_kv_heads=2, ffn=120, vocab=203, dtype="fp32")
# fewer K steps than the ring of the kernel for many rows is deep, ragged blocks of every projection
_SHORT = replace(_SMALL, d_model=192, n_q_heads=3, n_kv_heads=3, ffn=320, vocab=515)
_GROUPED = replace(_SMALL, d_model=1024, n_q_heads=8, n_kv_heads=1, head_dim=128)


@pytest.mark.parametrize("model,n", [(_SMALL, n) for n in (1, 16, 17, 32, 33, 64, 65, 128, 145, 256)]
                         + [(_WIDE, n) for n in (3, 16, 31, 64, 130)] + [(_GROUPED, n) for n in (2, 19, 70)] + [(_SHORT, n) for n in (65, 129)] + [(_FLOAT, n) for n in (1, 9, 16, 17)])
def test_decode_batches_of_few_rows(model, n):
    cfg = _GPT2S.with_(name="few_rows", model=model, n_samples=n, prompt_len=(3, 5), gain_jitter=0.05)
    ref = H.oracle_stage(cfg, n=n, max_len=4)
    got = H.run_gpu_stage(cfg, ref, fused=False, R_t=0, chunk_tokens=64)
    H.compare_stage(cfg, ref, got)


@pytest.mark.parametrize("model,n", [(_WIDE, 33), (_WIDE, 130), (_SMALL, 145), (_SHORT, 66)])
def test_decode_batches_read_half_copies(model, n):
    cfg = _GPT2S.with_(name="few_rows_half", model=model, n_samples=n, prompt_len=(3, 5), gain_jitter=0.05)
    ref = H.oracle_stage(cfg, n=n, max_len=4)
    got = H.run_gpu_stage(cfg, ref, fused=False, R_t=0, chunk_tokens=64, half_weight_copies=True)
    H.compare_stage(cfg, ref, got)


# one to eight weight blocks per workgroup (gate||up and head, up to 32 rows), ragged last workgroups; O and down in three and four planes,
# in blocks of two (N = 5120) and with a K that four waves do not share evenly
_BLOCKS7 = replace(_SMALL, n_layers=1, d_model=1088, n_q_heads=3, n_kv_heads=3, ffn=13760, vocab=31999)
_BLOCKS6 = replace(_BLOCKS7, ffn=10944, vocab=15351)
_PLANES = replace(_BLOCKS7, d_model=5120, n_q_heads=2, n_kv_heads=2, head_dim=128, ffn=3456, vocab=515)
_EIGHT_K = replace(_PLANES, d_model=8192, n_q_heads=1, n_kv_heads=1, ffn=6144)


@pytest.mark.parametrize("model,n", [(_BLOCKS7, 11), (_BLOCKS7, 29), (_BLOCKS6, 16), (_BLOCKS6, 17), (_PLANES, 1), (_PLANES, 9), (_PLANES, 32),
                                     (_EIGHT_K, 5), (_EIGHT_K, 33), (replace(_SMALL, vocab=32000), 50)])
def test_decode_batches_of_several_weight_blocks(model, n):
    cfg = _GPT2S.with_(name="few_rows_blocks", model=model, n_samples=n, prompt_len=(3, 5), gain_jitter=0.05)
    ref = H.oracle_stage(cfg, n=n, max_len=3)
    got = H.run_gpu_stage(cfg, ref, fused=False, R_t=0, chunk_tokens=64)
    H.compare_stage(cfg, ref, got)


# The shapes of real widths that the models above do not have: three to five weight blocks in rotary and planes, and seven
# (gate||up) and three (QKV) with 33 rows of 8192 columns.  A layer of such a width is too much for the oracle at these
# row counts, so decode steps are held to the Actor's own re-scoring pass, which runs on the kernels for many rows.
_7B, _13B, _70B = (CONFIGS[k].model for k in ("7b", "13b", "70b_slice"))
_2048 = replace(_7B, d_model=2048, n_q_heads=16, n_kv_heads=16, ffn=5504)


@pytest.mark.parametrize("model,n", [(_2048, 17), (_7B, 9), (_7B, 17), (_13B, 9), (_13B, 17), (_70B, 9), (_70B, 33), (_70B, 64)])
def test_decode_steps_of_real_widths_agree_with_scoring(model, n):
    cfg = _GPT2S.with_(name="real_width", model=replace(model, n_layers=1, vocab=4100), n_samples=n, prompt_len=(40, 44), gain_jitter=0.05)
    wl = make_workload(cfg, n)
    inp = {"prompt_tokens": wl["prompt_tokens"], "prompt_offsets": wl["prompt_offsets"], "n_layers": None,
           "out_len": np.minimum(wl["out_len"], 5).astype(np.int32), "weights": [make_weights(cfg, 0, device="cuda")]}
    got = H.run_gpu_stage(cfg, inp, fused=False, R_t=0, chunk_tokens=8192, role_mask=1, max_batch_tokens=8192)
    d = np.abs(got["lp_actor"].astype(np.float64) - got["lp_actor_rescored"])
    assert int(got["stats"].n_steps) >= 4 and float(np.abs(got["lp_actor"]).max()) > 5
    # the oracle's tolerance for log-probs on half activations; a wrong column or row is off by its own size (~8)
    assert float(d.max()) < H.LP_TOL["bf16"], d.max()
