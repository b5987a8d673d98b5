"""K splits of GEMMs beyond 256 rows: a split that leaves a plane without a K range (the plane is zero), and the
library's own splits of ragged shapes."""
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


@pytest.mark.parametrize("half_weights", [False, True])
@pytest.mark.parametrize("M,N,K", [(257, 1537, 1600), (300, 4100, 768), (511, 1100, 4096), (1000, 2052, 2048), (2100, 1284, 3456), (5000, 1300, 320)])
def test_ragged_tall_gemms_with_the_chosen_split(M, N, K, half_weights):
    """The stage's own kernel and K split on both sides of where they change, ragged in M and N."""
    import paper_2409_13221_amd as R
    g = torch.Generator().manual_seed(M + N + K)
    A = torch.randn(M, K, generator=g).half().cuda()
    W = (torch.randn(N, K, generator=g) * 0.02).to(torch.bfloat16).cuda()
    ns = R.rlhf_op_gemm_nsplit(R.RLHF_BF16, M, N, K, 8)
    out = torch.full((ns, M, N), float("nan"), device="cuda")
    R.rlhf_op_gemm(A, R.rlhf_op_bf16_to_half(W) if half_weights else W, out, ns)
    want = A.double() @ W.double().t()
    # float sums as above; weights below 2^-14 land on half's subnormal grid (up to 2^-24 each, activations of size 1)
    tol = 2.0 ** -23 * K ** 0.5 * float(want.abs().max()) + 2.0 ** -24 * K ** 0.5 * 4
    assert float((out.double().sum(0) - want).abs().max()) <= tol
