"""K splits of the compute-bound GEMM that leave a plane without a K range: the plane is zero."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("M,N,K,nsplit,variant", [(300, 2048, 128, 3, 0), (257, 1600, 64, 2, 0), (300, 520, 128, 3, 7), (700, 1544, 320, 4, 0)])
def test_tall_gemm_with_a_plane_without_k(act, M, N, K, nsplit, variant):
    import paper_2409_13221_amd as R
    g = torch.Generator().manual_seed(M + N)
    A = torch.randn(M, K, generator=g).to(act)
    W = (torch.randn(N, K, generator=g) * 0.02).to(torch.bfloat16)
    out = torch.full((nsplit, M, N), float("nan"), device="cuda")
    R.rlhf_op_gemm(A.cuda(), W.cuda(), out, nsplit, variant)
    torch.cuda.synchronize()
    want = A.double() @ W.double().T
    # exact inputs; float sums of K products of size 0.02: a few roundings of the largest partial sum
    np.testing.assert_allclose(out.double().sum(0).cpu().numpy(), want.numpy(), rtol=0, atol=2.0 ** -23 * K ** 0.5 * float(want.abs().max()))
