"""How many partial sums a product's elements are added up in is part of its result: a 256x256 tile and the square register-staged one run through k (of a
slice) in one chain of fp32 additions, the other kernels in two, and fewer chains round worse.  The choice of a kernel may not lower that number where
another kernel is faster; the shapes here are ones where a faster kernel with fewer chains is at hand."""
import pytest

from tests.test_abi_host import B  # noqa: F401  (fixture)

NN, NT, TN = "GEMM_NN", "GEMM_NT", "GEMM_TN"
OP, PASS = "oases_op_gemm_variant", "oases_pass_gemm_variant"


def chains(variant):
    """Partial sums of an element, from the kernel's name (1e8 W + 1e6 slices + 1e3 BM + BN)."""
    w, slices, bm, bn = variant // 100000000, variant // 1000000 % 100, variant // 1000 % 1000, variant % 1000
    assert w in (0, 1, 2, 3, 4, 5, 6)
    return slices * (1 if w == 0 or (w in (2, 3) and (bm, bn) == (256, 256)) else 2)


@pytest.mark.parametrize("query,op,epi,M,N,K,least", [
    (PASS, NT, "EPI_DSWIGLU", 8192, 1376, 4096, 2), (PASS, NN, "EPI_BIAS_GELU", 2120, 5120, 3840, 2), (PASS, NN, "EPI_BIAS_GELU", 2856, 3072, 768, 2),
    (PASS, NT, "EPI_DGELU", 6120, 1536, 768, 2), (PASS, NN, "EPI_F32", 8304, 4096, 512, 2), (PASS, NT, "EPI_DGELU", 9400, 1080, 208, 2),
    (PASS, NN, "EPI_SWIGLU", 15552, 6592, 576, 2), (PASS, NN, "EPI_BIAS_BF16", 1456, 5576, 1856, 2), (PASS, NT, "EPI_F32", 5888, 1840, 448, 2),
    (OP, NN, "EPI_F32", 8160, 5120, 2560, 2), (OP, NT, "EPI_F32", 7040, 3456, 3456, 2), (OP, NN, "EPI_F32", 7112, 3456, 4608, 2),
    (PASS, TN, "EPI_F32", 3584, 2688, 1072, 2), (PASS, TN, "EPI_F32", 3840, 3840, 2120, 2), (OP, TN, "EPI_F32", 3840, 3840, 2120, 2),
    (PASS, TN, "EPI_F32", 7384, 9232, 13128, 2), (OP, TN, "EPI_F32", 664, 6768, 96, 2), (PASS, TN, "EPI_F32", 1536, 3072, 11144, 8),
    (OP, TN, "EPI_F32", 1536, 3072, 11144, 8),
])
def test_partial_sums(B, query, op, epi, M, N, K, least):
    v = getattr(B.lib, query)(getattr(B, op), getattr(B, epi), M, N, K, 256 << 20)
    assert chains(v) >= least, v


@pytest.mark.parametrize("query,M,N,K,variant", [
    (OP, 6144, 3072, 7240, 601128256), (PASS, 3072, 3072, 2920, 601128256), (OP, 12336, 472, 1064, 601128256), (OP, 11544, 144, 4928, 602128256), (OP, 5728, 168, 6720, 604128256),
    (OP, 5728, 168, 6656, 304128256),      # whole slices
    (PASS, 15544, 136, 1248, 501128128),   # 122 tiles of 128x256 for 256 CUs
    (PASS, 6928, 408, 1240, 501128128),    # 110
    (PASS, 2560, 5120, 1016, 401064128),   # too few rows
    (PASS, 3072, 3072, 3072, 301256256),   # whole stages: as the model has it
])
def test_weight_gradients_over_ragged_rows(B, query, M, N, K, variant):
    """The 128x256 eight-wave kernel where it adds in the same order and is faster (K: rows, no whole number of 64-wide stages or of them a slice)."""
    assert getattr(B.lib, query)(B.GEMM_TN, B.EPI_F32, M, N, K, 256 << 20) == variant


@pytest.mark.parametrize("op,epi,M,N,K,variant", [(NT, "EPI_F32", 7040, 3456, 3456, 301128256), (NN, "EPI_BF16", 8648, 4736, 4096, 301128256), (TN, "EPI_F32", 14280, 1600, 5568, 301128256),
                                                  (NT, "EPI_DGELU", 8232, 832, 768, 101256128), (NN, "EPI_BIAS_BF16", 9056, 896, 384, 101256128)])
def test_ragged_rows_at_long_and_short_k(B, op, epi, M, N, K, variant):
    """256x128 register-staged tiles, and the eight-wave kernel that adds in the same order, from k = 2048 on."""
    assert B.lib.oases_pass_gemm_variant(getattr(B, op), getattr(B, epi), M, N, K, 256 << 20) == variant
