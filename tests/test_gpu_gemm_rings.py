"""The eight-wave GEMM kernels (variants 301256256 and 301128256) at the K where their rings of operand tiles can go wrong: fewer k tiles than a ring
holds, as many, one more, an odd number of them (the second half of the last 64-wide unit of a k-major operand lies beyond K), loops of one and of several
turns; each K on memory that holds NaN behind the operands' last k, so that whatever is multiplied too much shows."""
import pytest
import torch

from tests.test_gpu_ops import B, gen  # noqa: F401  (fixtures)
from tests.util import assert_bf16_close, bf16_round, dev, randn, rel_err

pytestmark = pytest.mark.gpu


def padded(x, rows, cols):
    """x on the device, inside a larger array of NaN: rows below it and columns beside it."""
    out = torch.full((x.shape[0] + rows, x.shape[1] + cols), float("nan"), dtype=torch.bfloat16, device="cuda")
    out[:x.shape[0], :x.shape[1]] = x.to(device="cuda", dtype=torch.bfloat16)
    return out


@pytest.mark.parametrize("op,variant,M,N", [("NN", 301256256, 256, 328), ("NT", 301256256, 512, 256), ("TN", 301256256, 264, 328),
                                            ("NN", 301128256, 136, 264), ("NT", 301128256, 72, 328), ("TN", 301128256, 200, 264)])
def test_rings(B, op, variant, M, N):
    """Exact products of bf16 values and fp32 sums against fp64: 1e-5; half a bf16 ulp for the bf16 output."""
    step = 32 if variant == 301256256 else 64
    for K in [step * n for n in (1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 16)]:
        g = gen(M + N + K)
        a, b = bf16_round(randn(g, M, K)), bf16_round(randn(g, K, N, scale=0.05))
        ref = a @ b
        ad = padded(a, 0, 64) if op != "TN" else padded(a.t(), 64, 0)
        bd = padded(b.t(), 0, 64) if op == "NT" else padded(b, 64, 0)
        opc = {"NN": B.GEMM_NN, "NT": B.GEMM_NT, "TN": B.GEMM_TN}[op]
        run = lambda epi, c: B.check(B.lib.oases_op_gemm_forced(variant, opc, epi, M, N, K, ad.data_ptr(), ad.shape[1], bd.data_ptr(), bd.shape[1], c.data_ptr(), N,
                                                                None, None, 0, None, 0, None))
        c0 = randn(g, M, N).float()
        c = dev(c0, torch.float32)
        run(B.EPI_F32, c)
        assert rel_err(c.cpu().double(), ref + (c0.double() if op == "TN" else 0.0)) < 1e-5, K
        if op != "TN":
            cb = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
            run(B.EPI_BF16, cb)
            assert_bf16_close(cb.float(), ref, 1e-5, 2e-6 * float(ref.abs().max()), f"{op} {K}")
