"""Greedy pick of one plane of logits in one kernel: column counts at the edges of its per-thread counts and just beyond
them (two kernels again), ties at both ends of a row, imposed tokens, a row without a finite maximum."""
import numpy as np
import pytest
import torch

import paper_2409_13221_amd as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [2, 1023, 1024, 1025, 4096, 4097, 16384, 16385, 32768, 32769])
def test_one_plane_of_logits(vocab):
    rows = 5
    z = torch.randn(rows, vocab, device="cuda") * 3
    top = float(z.max()) + 1
    z[0, 0] = z[0, -1] = top                               # the lowest id wins
    z[1, -1] = top
    z[2, vocab // 2] = z[2, -1] = top
    z[4] = float("-inf")
    forced = torch.tensor([-1, -1, -1, vocab - 1, -1], dtype=torch.int32, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    lp = torch.zeros(rows, device="cuda")
    dst = torch.arange(rows, dtype=torch.int32, device="cuda")
    picked = torch.zeros(rows, dtype=torch.int32, device="cuda")
    scratch = torch.zeros(R.lib().rlhf_op_pick_scratch_floats(rows), device="cuda")
    rc = R.lib().rlhf_op_pick(z.data_ptr(), 1, 0, rows, vocab, forced.data_ptr(), tokens.data_ptr(), dst.data_ptr(), lp.data_ptr(),
                              dst.data_ptr(), picked.data_ptr(), scratch.data_ptr(), None)
    assert rc == 0
    torch.cuda.synchronize()
    want = [0, vocab - 1, vocab // 2, vocab - 1]
    assert tokens.tolist()[:4] == want and picked.tolist()[:4] == want
    assert 0 <= tokens.tolist()[4] < vocab and not np.isfinite(float(lp[4]))
    ref = torch.log_softmax(z[:4].double(), -1).cpu().numpy()[np.arange(4), want]
    # 32 terms a thread, then 1024 of them, each rounded to 24 bits; log-probs of size up to ~20
    np.testing.assert_allclose(lp[:4].cpu().numpy(), ref, rtol=0, atol=1e-5)
