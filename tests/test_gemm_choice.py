"""K splits that the library chooses for passes beyond 256 rows, at shapes where kernels and splits are far apart
(microseconds measured on an MI355X, projection and the RMSNorm behind it, bf16 weights)."""
import pytest

import paper_2409_13221_amd as R


@pytest.mark.parametrize("M,N,K,nsplit", [
    (300, 1536, 1536, 4),     # 128 x 128 tiles 20.7; 256 x 256 tiles 26.5 with 6 to 8 splits, 50 unsplit
    (257, 768, 2048, 8),      # 128 x 128 tiles 16.0
    (512, 2048, 2048, 4),     # 128 x 128 tiles 27.4
    (2048, 1280, 3456, 4),    # 256 x 256 tiles 48.5, 90 unsplit; 128 x 128 tiles 56.0 with 2 splits
    (3072, 1280, 3456, 2),    # 256 x 256 tiles 62.7; 128 x 128 tiles 82.7
    (3072, 1536, 1536, 2),    # 256 x 256 tiles 45.4, 57.8 unsplit; 128 x 128 tiles 54.4
    (8192, 1280, 3456, 1),    # 256 x 256 tiles 120; 128 x 128 tiles 170
    (8192, 4096, 4096, 1),
])
def test_split_of_passes_beyond_256_rows(M, N, K, nsplit):
    assert R.rlhf_op_gemm_nsplit(R.RLHF_BF16, M, N, K, 16) == nsplit


@pytest.mark.parametrize("max_split", [1, 2, 3, 5, 16])
def test_every_split_has_a_k_range(max_split):
    for M in (129, 257, 300, 511, 512, 2048, 20000):
        for N in (64, 1024, 1088, 1536, 4095, 4096, 12288):
            for K in (64, 72, 128, 320, 1088, 4096):
                ns = R.rlhf_op_gemm_nsplit(R.RLHF_BF16, M, N, K, max_split)
                assert 1 <= ns <= max_split
                assert (ns - 1) * (-(-(-(-K // ns)) // 64) * 64) < K


@pytest.mark.parametrize("M,N,K,nsplit", [
    (64, 1024, 1024, 16),     # planes 7, unsplit 31
    (512, 1024, 1024, 8),     # planes 22, unsplit 37
    (512, 4096, 4096, 1),     # planes 238 with their reading, unsplit 174
    (256, 4096, 4096, 4),     # planes 133, unsplit 142
    (256, 11008, 2048, 1),    # planes 176, unsplit 122
    (460, 4096, 256, 1),      # planes 24, unsplit 15
])
def test_split_of_float_models(M, N, K, nsplit):
    assert R.rlhf_op_gemm_nsplit(R.RLHF_FP32, M, N, K, 16) == nsplit
