"""fp32 results with a leading dimension beyond what 32-bit offsets within 16 rows reach (35.8 million columns): every kernel that stores them in whole lines,
bit for bit what it gives with a narrow C."""
import pytest
import torch

from tests.test_gpu_ops import B, gen  # noqa: F401  (fixtures)
from tests.util import randn

pytestmark = pytest.mark.gpu
WIDE = 36_000_000


@pytest.fixture(scope="module")
def memory():
    yield torch.empty(256 * WIDE, device="cuda")     # 37 GB, of which the tests touch a few columns
    torch.cuda.empty_cache()


def operands(M, N, K, seed):
    return randn(gen(seed), M, K).bfloat16().cuda(), randn(gen(seed + 1), K, N).bfloat16().cuda()


@pytest.mark.parametrize("op,variant,M,N,K", [("NN", 301256256, 256, 256, 128), ("NT", 301256256, 256, 256, 128), ("TN", 301256256, 256, 256, 128), ("NN", 301128256, 128, 256, 128),
                                              ("NT", 301128256, 128, 256, 128), ("TN", 301128256, 128, 256, 128), ("TN", 302128256, 128, 256, 256), ("TN", 601128256, 128, 256, 1032),
                                              ("NN", 401064064, 64, 64, 128), ("NT", 401064128, 64, 128, 128), ("TN", 401064128, 64, 128, 128), ("TN", 501128128, 128, 128, 128)])
def test_wide_result(B, memory, op, variant, M, N, K):
    a, b = operands(M, N, K, M + K)
    ad, bd = (a.t().contiguous() if op == "TN" else a), (b.t().contiguous() if op == "NT" else b)
    opc = {"NN": B.GEMM_NN, "NT": B.GEMM_NT, "TN": B.GEMM_TN}[op]
    ws = torch.empty(8 << 20, dtype=torch.uint8, device="cuda")
    start = torch.randn(M, N, device="cuda")
    narrow, wide = start.clone(), memory.as_strided((M, N), (WIDE, 1))
    wide.copy_(start)
    beyond = memory.as_strided((M, 8), (WIDE, 1), N).fill_(7.0)
    for c, ldc in ((narrow, N), (wide, WIDE)):
        B.check(B.lib.oases_op_gemm_forced(variant, opc, B.EPI_F32, M, N, K, ad.data_ptr(), ad.shape[1], bd.data_ptr(), bd.shape[1], c.data_ptr(), ldc, None, None, 0,
                                           ws.data_ptr(), ws.numel(), None))
    assert torch.equal(narrow, wide) and bool((beyond == 7.0).all())
    assert not torch.equal(narrow, start)


@pytest.mark.parametrize("variant", [None, 301128256, 302128256, 401064128])
def test_two_in_a_launch(B, memory, variant):
    """variant None: oases_op_gemm_tn_pair."""
    M, N, K = 128, 256, 256
    ws = torch.empty(8 << 20, dtype=torch.uint8, device="cuda")
    ops = [[x.contiguous() for x in (a.t(), b)] for a, b in (operands(M, N, K, 1), operands(M, N, K, 3))]
    results = []
    for first, ld0 in ((torch.ones(M, N, device="cuda"), N), (memory.as_strided((M, N), (WIDE, 1)).fill_(1.0), WIDE)):
        second = torch.ones(M, N, device="cuda")
        args = [K]
        for (a, b), c, ld in ((ops[0], first, ld0), (ops[1], second, N)):
            args += [M, N, a.data_ptr(), M, b.data_ptr(), N, c.data_ptr(), ld]
        B.check(B.lib.oases_op_gemm_tn_pair(*args, None) if variant is None else B.lib.oases_op_gemm_tn_group(variant, *args, ws.data_ptr(), ws.numel(), None))
        results.append((first, second))
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])
