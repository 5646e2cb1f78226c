"""The bf16 epilogues of the large-tile GEMM kernels, which read and write eight columns of a row at a time: rows of C and aux
that start at odd multiples of 8 bytes, operands that end eight columns into a 32-column tile or a few rows into the last tile."""
import pytest
import torch

from tests.test_gpu_ops import B, gen, lo  # noqa: F401  (fixtures)
from tests.test_gpu_gemm_small import operands
from tests.test_gpu_ops_llama import interleave, ll  # noqa: F401
from tests.util import assert_bf16_close, bf16_round, dev, randn

pytestmark = pytest.mark.gpu

# eight-wave 256 x 256 and 128 x 256, four-wave 128 x 256, register-staged kernels
CASES = [(301256256, "NN", 256, 264, 128), (301256256, "NT", 512, 256, 64), (301128256, "NN", 136, 264, 192), (301128256, "NT", 128, 280, 64),
         (301128256, "NT", 136, 264, 192),
         (201128256, "NT", 136, 264, 128), (1256256, "NN", 264, 296, 72), (1128128, "NT", 136, 152, 72)]


@pytest.mark.parametrize("variant,op,M,N,K", CASES)
def test_bf16_epilogues(B, lo, variant, op, M, N, K):
    """Tolerances as for the small tiles: half a bf16 ulp plus the error of fp32 sums and of the fast exponentials."""
    g = gen(M + N + K)
    ref, ad, bd, opc, lda, ldb = operands(B, op, M, N, K, g)
    bias, ld = dev(0.1 * randn(g, N), torch.float32), N + 4
    pre = torch.full((M, ld), 7.0, dtype=torch.bfloat16, device="cuda")
    pre[:, :N] = dev(bf16_round(randn(g, M, N)), torch.bfloat16)
    z = ref + bias.cpu().double()
    cases = [(B.EPI_BF16, ref, 2e-6 * float(ref.abs().max())), (B.EPI_BIAS_BF16, z, 2e-6 * float(z.abs().max())),
             (B.EPI_BIAS_GELU, lo.gelu_fwd(z), 1e-5), (B.EPI_DGELU, ref * lo.gelu_grad(pre[:, :N].float().cpu().double()), 1e-5)]
    for epi, want, atol in cases:
        if epi in (B.EPI_BIAS_BF16, B.EPI_BIAS_GELU) and op != "NN" or epi == B.EPI_DGELU and op != "NT":
            continue
        c = torch.full((M + 2, ld), 7.0, dtype=torch.bfloat16, device="cuda")
        aux = torch.full((M + 2, ld), 7.0, dtype=torch.bfloat16, device="cuda") if epi == B.EPI_BIAS_GELU else pre
        B.check(B.lib.oases_op_gemm_forced(variant, opc, epi, M, N, K, ad.data_ptr(), lda, bd.data_ptr(), ldb, c.data_ptr(), ld,
                                           bias.data_ptr(), aux.data_ptr(), ld, None, 0, None))
        assert_bf16_close(c[:M, :N].float(), want, 1e-4 if atol == 1e-5 else 1e-5, atol, f"{epi} {variant}")
        assert bool((c[:M, N:] == 7.0).all()) and bool((c[M:] == 7.0).all())
        if epi == B.EPI_BIAS_GELU:
            assert_bf16_close(aux[:M, :N].float(), z, 1e-5, 2e-6 * float(z.abs().max()))
            assert bool((aux[:M, N:] == 7.0).all()) and bool((aux[M:] == 7.0).all())


@pytest.mark.parametrize("variant,M,fp,K", [(301256256, 256, 160, 64), (301128256, 136, 96, 128), (1256256, 264, 160, 72)])
def test_swiglu_epilogues(B, ll, variant, M, fp, K):
    g = gen(M + fp + K)
    a, wg, wu = bf16_round(randn(g, M, K)), bf16_round(randn(g, K, fp, scale=0.05)), bf16_round(randn(g, K, fp, scale=0.05))
    ad, wd = dev(a, torch.bfloat16), dev(interleave(wg, wu), torch.bfloat16)
    f, gu, dgu = (torch.full((M + 2, n + 4), 7.0, dtype=torch.bfloat16, device="cuda") for n in (fp, 2 * fp, 2 * fp))
    B.check(B.lib.oases_op_gemm_forced(variant, B.GEMM_NN, B.EPI_SWIGLU, M, 2 * fp, K, ad.data_ptr(), K, wd.data_ptr(), 2 * fp, f.data_ptr(), fp + 4,
                                       None, gu.data_ptr(), 2 * fp + 4, None, 0, None))
    gate, up = a.double() @ wg.double(), a.double() @ wu.double()
    assert_bf16_close(gu[:M, :2 * fp].float(), interleave(gate, up), 1e-5, 2e-6 * float(gate.abs().max()))
    assert_bf16_close(f[:M, :fp].float(), ll.silu(gate) * up, 1e-4, 1e-5)
    assert all(bool((t[:M, n:] == 7.0).all()) and bool((t[M:] == 7.0).all()) for t, n in ((f, fp), (gu, 2 * fp)))
    w2 = bf16_round(randn(g, fp, K, scale=0.05))
    w2d = dev(w2, torch.bfloat16)
    dF = a.double() @ w2.double().t()
    gs = gu[:M, :2 * fp].float().cpu().double().reshape(M, fp // 32, 2, 32)
    gst, ust = gs[:, :, 0].reshape(M, fp), gs[:, :, 1].reshape(M, fp)
    dvariant = 301128256 if variant == 301256256 else variant      # NT on 256 x 256 eight-wave tiles needs whole tiles
    B.check(B.lib.oases_op_gemm_forced(dvariant, B.GEMM_NT, B.EPI_DSWIGLU, M, fp, K, ad.data_ptr(), K, w2d.data_ptr(), K, dgu.data_ptr(), 2 * fp + 4, None,
                                       gu.data_ptr(), 2 * fp + 4, None, 0, None))
    assert_bf16_close(dgu[:M, :2 * fp].float(), interleave(dF * ust * ll.silu_grad(gst), dF * ll.silu(gst)), 1e-4, 1e-5)
    assert bool((dgu[:M, 2 * fp:] == 7.0).all()) and bool((dgu[M:] == 7.0).all())
