"""The small-tile GEMM kernels (variants 4SS064064, 4SS064128 and 5SS128128) at the sizes where they can go wrong: fewer k tiles than LDS
stages, as many, more; k tails; operands that end inside the only or the last tile; k slices, the last one shorter."""
import pytest
import torch

from tests.test_gpu_ops import B, gen, lo  # noqa: F401  (fixtures)
from tests.test_gpu_ops_llama import interleave, ll  # noqa: F401
from tests.util import assert_bf16_close, bf16_round, dev, randn, rel_err

pytestmark = pytest.mark.gpu

# (M, N, K): one 8 x 8 corner, one whole tile, ragged tiles with a k tail, K one stage short of / equal to / beyond the stages
SHAPES = [(8, 8, 8), (64, 128, 64), (72, 136, 72), (200, 264, 600), (136, 72, 192), (64, 64, 320), (128, 256, 384), (264, 392, 1096)]


def operands(B, op, M, N, K, g):
    a, b = bf16_round(randn(g, M, K)), bf16_round(randn(g, K, N, scale=0.05))
    ad = dev(a if op != "TN" else a.t().contiguous(), torch.bfloat16)
    bd = dev(b if op != "NT" else b.t().contiguous(), torch.bfloat16)
    opc = {"NN": B.GEMM_NN, "NT": B.GEMM_NT, "TN": B.GEMM_TN}[op]
    return a @ b, ad, bd, opc, (K if op != "TN" else M), (N if op != "NT" else K)


@pytest.mark.parametrize("variant", [401064064, 401064128, 402064064, 403064128, 501128128, 503128128])
@pytest.mark.parametrize("op", ["NN", "NT", "TN"])
def test_small_tiles(B, lo, op, variant):
    """fp32 output (accumulated into for TN) inside a larger buffer that must stay as it was, then the fused epilogues.
    Tolerances: exact products of bf16 values and fp32 sums against fp64 (1e-5); half a bf16 ulp for bf16 outputs."""
    S = variant // 1000000 % 100
    for M, N, K in SHAPES:
        if S > 1 and (S - 1) * (-(-(-(-K // S)) // 64) * 64) >= K:
            continue                                        # a slice would be empty: refused, tested below
        g = gen(M + N + K + S)
        ref, ad, bd, opc, lda, ldb = operands(B, op, M, N, K, g)
        ws = torch.full((S * M * N * 4,), 0xFF, dtype=torch.uint8, device="cuda")
        ldc, guard = N + 12, 3
        c0 = randn(g, M + 2 * guard, ldc).float()
        c = dev(c0, torch.float32)
        B.check(B.lib.oases_op_gemm_forced(variant, opc, B.EPI_F32, M, N, K, ad.data_ptr(), lda, bd.data_ptr(), ldb, c.data_ptr() + guard * ldc * 4, ldc,
                                           None, None, 0, ws.data_ptr(), ws.numel(), None))
        out = c.cpu()
        body = out[guard:guard + M].double()
        assert rel_err(body[:, :N], ref + (c0[guard:guard + M, :N].double() if op == "TN" else 0.0)) < 1e-5, (M, N, K)
        assert torch.equal(body[:, N:], c0[guard:guard + M, N:].double())
        assert torch.equal(out[:guard], c0[:guard]) and torch.equal(out[guard + M:], c0[guard + M:])
        if op == "TN":
            continue
        bias = dev(0.1 * randn(g, N), torch.float32)
        pre = dev(bf16_round(randn(g, M, N)), torch.bfloat16)
        z = ref + bias.cpu().double()
        run = lambda epi, c, auxp: B.check(B.lib.oases_op_gemm_forced(variant, opc, epi, M, N, K, ad.data_ptr(), lda, bd.data_ptr(), ldb, c.data_ptr(), N + 8,
                                                                      bias.data_ptr(), auxp, N, ws.data_ptr(), ws.numel(), None))
        for epi, want, atol in ((B.EPI_BF16, ref, 2e-6 * float(ref.abs().max())), (B.EPI_BIAS_BF16, z, 2e-6 * float(z.abs().max())),
                                (B.EPI_BIAS_GELU, lo.gelu_fwd(z), 1e-5), (B.EPI_DGELU, ref * lo.gelu_grad(pre.float().cpu().double()), 1e-5)):
            cb = torch.full((M, N + 8), 7.0, dtype=torch.bfloat16, device="cuda")
            aux = torch.empty(M, N, dtype=torch.bfloat16, device="cuda") if epi == B.EPI_BIAS_GELU else pre
            run(epi, cb, aux.data_ptr())
            assert_bf16_close(cb[:, :N].float(), want, 1e-4 if atol == 1e-5 else 1e-5, atol, f"{epi} {M} {N} {K}")
            assert bool((cb[:, N:] == 7.0).all())
            if epi == B.EPI_BIAS_GELU:
                assert_bf16_close(aux.float(), z, 1e-5, 2e-6 * float(z.abs().max()))


@pytest.mark.parametrize("M,fp,K", [(8, 32, 8), (72, 96, 328), (200, 352, 704)])
def test_small_tiles_swiglu(B, ll, M, fp, K):
    g = gen(M + fp + K)
    a, wg, wu = bf16_round(randn(g, M, K)), bf16_round(randn(g, K, fp, scale=0.05)), bf16_round(randn(g, K, fp, scale=0.05))
    ad, wd = dev(a, torch.bfloat16), dev(interleave(wg, wu), torch.bfloat16)
    gate, up = a.double() @ wg.double(), a.double() @ wu.double()
    for variant in (401064064, 401064128, 501128128):
        f = torch.full((M, fp + 8), 7.0, dtype=torch.bfloat16, device="cuda")
        gu = torch.full((M, 2 * fp + 8), 7.0, dtype=torch.bfloat16, device="cuda")
        fwd = (B.GEMM_NN, B.EPI_SWIGLU, M, 2 * fp, K, ad.data_ptr(), K, wd.data_ptr(), 2 * fp, f.data_ptr(), fp + 8, None, gu.data_ptr(), 2 * fp + 8, None, 0, None)
        if variant == 401064064:
            assert B.lib.oases_op_gemm_forced(variant, *fwd) == B.EINVAL     # gate and up columns must meet in one wave
            continue
        B.check(B.lib.oases_op_gemm_forced(variant, *fwd))
        assert_bf16_close(gu[:, :2 * fp].float(), interleave(gate, up), 1e-5, 2e-6 * float(gate.abs().max()))
        assert_bf16_close(f[:, :fp].float(), ll.silu(gate) * up, 1e-4, 1e-5)
        assert bool((f[:, fp:] == 7.0).all()) and bool((gu[:, 2 * fp:] == 7.0).all())
    w2 = bf16_round(randn(g, fp, K, scale=0.05))
    w2d = dev(w2, torch.bfloat16)
    dF = a.double() @ w2.double().t()
    gs = gu[:, :2 * fp].float().cpu().double().reshape(M, fp // 32, 2, 32)
    gst, ust = gs[:, :, 0].reshape(M, fp), gs[:, :, 1].reshape(M, fp)
    for variant in (401064064, 401064128, 501128128):
        dgu = torch.full((M, 2 * fp + 8), 7.0, dtype=torch.bfloat16, device="cuda")
        B.check(B.lib.oases_op_gemm_forced(variant, B.GEMM_NT, B.EPI_DSWIGLU, M, fp, K, ad.data_ptr(), K, w2d.data_ptr(), K, dgu.data_ptr(), 2 * fp + 8, None,
                                           gu.data_ptr(), 2 * fp + 8, None, 0, None))
        assert_bf16_close(dgu[:, :2 * fp].float(), interleave(dF * ust * ll.silu_grad(gst), dF * ll.silu(gst)), 1e-4, 1e-5)
        assert bool((dgu[:, 2 * fp:] == 7.0).all())


def test_small_tiles_refusals_and_span(B):
    """Slices that would be empty, workspaces that are too small, operands of 2 GiB span: refused before any launch; the
    library's own choice then runs the register-staged kernel."""
    M, N, K, lda = 128, 64, 128, 1 << 23
    g = gen(5)
    a, b = bf16_round(randn(g, M, K)), bf16_round(randn(g, K, N, scale=0.05))
    ad, bd = dev(a, torch.bfloat16), dev(b, torch.bfloat16)
    c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    args = lambda A, ld, wsb: (B.GEMM_NN, B.EPI_F32, M, N, K, A.data_ptr(), ld, bd.data_ptr(), N, c.data_ptr(), N, None, None, 0, ws.data_ptr(), wsb, None)
    assert B.lib.oases_op_gemm_variant(B.GEMM_NN, B.EPI_F32, M, N, K, 0) == 401064064
    for v, wsb in ((403064064, 1 << 20), (402064064, 2 * M * N * 4 - 4), (417064064, 1 << 20), (401128128, 1 << 20), (501064064, 1 << 20)):
        assert B.lib.oases_op_gemm_forced(v, *args(ad, K, wsb)) == B.EINVAL, v
    big = torch.zeros(M, lda, dtype=torch.bfloat16, device="cuda")
    big[:, :K] = ad
    assert B.lib.oases_op_gemm_forced(401064064, *args(big, lda, 0)) == B.EINVAL
    B.check(B.lib.oases_op_gemm(*args(big, lda, 0)))
    torch.cuda.synchronize()
    assert rel_err(c, a @ b) < 1e-5
    del big
    torch.cuda.empty_cache()
