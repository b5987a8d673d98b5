"""Decode attention with enough rows for eight waves per workgroup (256 workgroups), each fetching a page ahead, and for
four waves (512): contexts at the edges of a page and of one, two and three pages per wave, and splits without pages."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import paper_2409_13221_amd as R
from tests import stage_harness as H
from tests.test_gpu_ops import _paged_case
from workload import CONFIGS

pytestmark = pytest.mark.gpu

_EDGES = [1, 2, 15, 16, 17, 127, 128, 129, 143, 144, 145, 255, 256, 257, 271, 272, 383, 384, 385, 400, 513]


@pytest.mark.parametrize("dtype,hd", [("half", 128), ("half", 64), ("bf16", 128), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("nsplit", [1, 2])
@pytest.mark.parametrize("heads", [3, 6])
def test_many_rows_of_uneven_contexts(dtype, hd, nsplit, heads):
    _compare(dtype, hd, nsplit, heads, [_EDGES[i % len(_EDGES)] for i in range(86)])


# four waves a row: every wave's first, second and third page, and the wave counts at which some have none
@pytest.mark.parametrize("dtype,hd", [("half", 128), ("half", 64), ("bf16", 128), ("fp32", 64), ("fp32", 128)])
def test_rows_of_short_contexts(dtype, hd):
    edges = [1, 16, 17, 48, 49, 64, 65, 80, 128, 129, 176, 177, 192, 193]
    _compare(dtype, hd, 1, 4, [edges[i % len(edges)] for i in range(128)])


def _compare(dtype, hd, nsplit, heads, ctx_lens):
    rows, n_layers, layer = len(ctx_lens), 2, 1
    q, pool, pt, rs, want = _paged_case(31, rows, heads, heads, hd, n_layers, layer, ctx_lens, dtype)
    qd, pd = q.cuda().reshape(rows, heads * hd).contiguous(), pool.cuda().contiguous()
    out = torch.zeros_like(qd)
    pa = torch.zeros(rows * heads * nsplit * hd, device="cuda")
    pm = torch.zeros(rows * heads * nsplit * 2, device="cuda")
    R.rlhf_op_paged_decode_attention(qd, pd, torch.from_numpy(pt).cuda(), torch.from_numpy(rs).cuda(),
                                     torch.tensor(ctx_lens, dtype=torch.int32).cuda(), out, pa, pm, layer, nsplit, n_layers,
                                     heads, heads, hd)
    torch.cuda.synchronize()
    # outputs are averages of values of size ~3 (a context of one token: the value itself), rounded to the type
    tol = {"bf16": 2e-2, "half": 3e-3, "fp32": 2e-5}[dtype]
    np.testing.assert_allclose(out.double().cpu().numpy().reshape(rows, heads, hd), want, rtol=0, atol=tol)


# 512 workgroups whose longest context passes from twelve pages to thirteen: four waves a row, then eight
def test_steps_across_the_longest_short_context():
    base = CONFIGS["gpt2s"]
    model = replace(base.model, n_layers=1, d_model=64, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn=64, vocab=203)
    cfg = base.with_(name="short_contexts", model=model, n_samples=128, prompt_len=(188, 190), gain_jitter=0.05)
    ref = H.oracle_stage(cfg, n=128, max_len=6)
    got = H.run_gpu_stage(cfg, ref, fused=False, R_t=0, chunk_tokens=4096, max_batch_tokens=4096)
    H.compare_stage(cfg, ref, got)
