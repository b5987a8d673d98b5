"""Decode attention with enough rows for eight waves per workgroup (256 workgroups), each fetching a page ahead:
contexts at the edges of a page and of one, two and three pages per wave, and splits without pages."""
import numpy as np
import pytest
import torch

import paper_2409_13221_amd as R
from tests.test_gpu_ops import _paged_case

pytestmark = pytest.mark.gpu

_EDGES = [1, 2, 15, 16, 17, 127, 128, 129, 143, 144, 145, 255, 256, 257, 271, 272, 383, 384, 385, 400, 513]


@pytest.mark.parametrize("dtype,hd", [("half", 128), ("half", 64), ("bf16", 128), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("nsplit", [1, 2])
def test_many_rows_of_uneven_contexts(dtype, hd, nsplit):
    ctx_lens = [_EDGES[i % len(_EDGES)] for i in range(86)]
    rows, heads, n_layers, layer = len(ctx_lens), 3, 2, 1
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
