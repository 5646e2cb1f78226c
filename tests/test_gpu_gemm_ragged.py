"""Products whose rows are no whole tiles of the eight-wave kernels: k-major operands that end inside a tile, and weight gradients over a number of
rows that is no whole number of k tiles (the last tile of a wave group partly or wholly beyond K, alone and two in a launch) or of slices.
The library's choice goes to those kernels here; memory behind the operands holds NaN."""
import pytest
import torch

from tests.test_gpu_gemm_rings import padded
from tests.test_gpu_ops import B, gen, lo  # noqa: F401  (fixtures)
from tests.util import assert_bf16_close, bf16_round, dev, randn, rel_err

pytestmark = pytest.mark.gpu
WS = 256 << 20


# the last two: k slices whose last one is shorter (2688 and 2624 rows; three times 1600 and 1408), added up by a second launch
@pytest.mark.parametrize("op,M,N,K,variant", [("NN", 6072, 4096, 448, 301128256), ("NT", 6072, 4096, 448, 301128256), ("NT", 4088, 4088, 256, 301128256),
                                                               ("TN", 1160, 4104, 1064, 601128256), ("TN", 2048, 4096, 2056, 601128256), ("TN", 2048, 4096, 2040, 601128256),
                                                               ("TN", 4096, 4096, 1048, 601128256), ("TN", 4096, 4088, 1080, 601128256), ("TN", 4088, 4096, 1992, 601128256),
                                                               ("TN", 11160, 136, 5312, 602128256), ("TN", 80, 8632, 6208, 604128256)])
def test_choice_of_ragged_rows(B, op, M, N, K, variant):
    """Exact products of bf16 values and fp32 sums against fp64: 1e-5; half a bf16 ulp for the bf16 output."""
    opc = {"NN": B.GEMM_NN, "NT": B.GEMM_NT, "TN": B.GEMM_TN}[op]
    assert B.lib.oases_op_gemm_variant(opc, B.EPI_F32, M, N, K, WS) == variant
    g = gen(M + N + K)
    a, b = bf16_round(randn(g, M, K)), bf16_round(randn(g, K, N, scale=0.05))
    ref = (a.cuda() @ b.cuda()).cpu()
    ad = padded(a, 0, 64) if op != "TN" else padded(a.t(), 64, 0)
    bd = padded(b.t(), 0, 64) if op == "NT" else padded(b, 64, 0)
    ws = torch.empty(WS, dtype=torch.uint8, device="cuda")
    run = lambda epi, c: B.check(B.lib.oases_op_gemm(opc, epi, M, N, K, ad.data_ptr(), ad.shape[1], bd.data_ptr(), bd.shape[1], c.data_ptr(), N, None, None, 0,
                                                     ws.data_ptr(), ws.numel(), None))
    c0 = randn(g, M, N).float()
    c = dev(c0, torch.float32)
    run(B.EPI_F32, c)
    assert rel_err(c.cpu().double(), ref + (c0.double() if op == "TN" else 0.0)) < 1e-5
    # the kernel that the query names can be forced, and is the one that the library takes
    cf = dev(c0, torch.float32)
    forced = lambda v: B.lib.oases_op_gemm_forced(v, opc, B.EPI_F32, M, N, K, ad.data_ptr(), ad.shape[1], bd.data_ptr(), bd.shape[1], cf.data_ptr(), N, None, None, 0,
                                                  ws.data_ptr(), ws.numel(), None)
    if op == "TN":
        assert forced(variant - 300000000) == B.EINVAL
    B.check(forced(variant))
    assert torch.equal(c, cf)
    if op != "TN":
        cb = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
        run(B.EPI_BF16, cb)
        assert_bf16_close(cb.float(), ref, 1e-5, 2e-6 * float(ref.abs().max()), op)


@pytest.mark.parametrize("seq,batch", [(1032, 1), (520, 3), (680, 3), (1064, 2), (1352, 3)])
def test_step_of_ragged_rows(B, lo, seq, batch):
    """A training step of a layer of 2048 over such rows: what the FFN products and their epilogues leave, and the weight gradients (in one launch or two), against
    the products of the pass's own operands in fp64."""
    from paper_2305_16121_amd import binding as Bi
    cfg = dict(hidden=2048, n_heads=16, seq=seq, batch=batch, tp=2, n_sub=1, n_layers=1, causal=1, dropout_p=0.0)
    H = Bi.Handle(Bi.make_cfg(cfg, rank=1))
    h, hp, fp, M = 2048, 1024, 4096, seq * batch
    g = torch.Generator(device="cuda").manual_seed(seq)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    w = {k: (n(*s) * 0.02).bfloat16() for k, s in dict(wqkv=(h, 3 * hp), wo=(hp, h), w1=(h, fp), w2=(fp, h)).items()}
    w.update({k: n(s) * 0.02 + (1.0 if k.endswith("_g") else 0.0) for k, s in dict(ln1_g=h, ln2_g=h, ln1_b=h, ln2_b=h, bqkv=3 * hp, bo=h, b1=fp, b2=h).items()})
    x, dy = n(M, h), n(M, h)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    grads = Bi.zero_grads_like(w)
    ws = torch.empty(H.workspace_bytes, dtype=torch.uint8, device="cuda")
    H.forward([w], x, y, ws)
    H.backward([w], x, dy, dx, [grads], ws)
    torch.cuda.synchronize()

    def t(name, cols):
        off, nb = H.tensor_span(name, 0)
        return ws[off:off + nb].view(torch.bfloat16).view(M, cols).double()

    z = t("v2", h) @ w["w1"].double() + w["b1"].double()
    assert_bf16_close(t("pre", fp).float(), z.cpu(), 1e-5, 2e-6 * float(z.abs().max()), "pre")
    assert_bf16_close(t("f", fp).float(), lo.gelu_fwd(z.cpu()), 1e-4, 1e-5, "f")
    df = t("dz2", h) @ w["w2"].double().t().contiguous()
    assert_bf16_close(t("dg", fp).float(), (df.cpu() * lo.gelu_grad(t("pre", fp).cpu())), 1e-4, 1e-5, "dg")
    for k, a, ca, b, cb in (("wqkv", "u", h, "dqkv", 3 * hp), ("wo", "attn", hp, "dz1", h), ("w1", "v2", h, "dg", fp), ("w2", "f", fp, "dz2", h)):
        ref = t(a, ca).t().contiguous() @ t(b, cb)
        assert rel_err(grads[k].double(), ref) < 2e-5, k


@pytest.mark.parametrize("K", [1032, 1064, 2040])
@pytest.mark.parametrize("M0,N0,M1,N1", [(256, 512, 128, 256), (136, 264, 8, 1000)])
def test_two_in_a_launch(B, K, M0, N0, M1, N1):
    """601128256 on two weight gradients over such rows, against the products in fp64 (the bound of the whole-stage test) and, bit for bit, each by itself."""
    ws = torch.full((64 << 20,), 0xFF, dtype=torch.uint8, device="cuda")
    sizes, c, old = ((M0, N0), (M1, N1)), [], []
    ab = [(padded(randn(gen(K + i), K, M).bfloat16(), 64, 0), padded(randn(gen(M + i), K, N).bfloat16(), 64, 0)) for i, (M, N) in enumerate(sizes)]
    args = lambda v: [v, K] + [x for i, (M, N) in enumerate(sizes) for x in (M, N, ab[i][0].data_ptr(), ab[i][0].shape[1], ab[i][1].data_ptr(), ab[i][1].shape[1], c[i].data_ptr(), N)]
    for i, (M, N) in enumerate(sizes):
        old.append(torch.randn(M, N, device="cuda"))
        c.append(old[i].clone())
    assert B.lib.oases_op_gemm_tn_group(*args(301128256), ws.data_ptr(), ws.numel(), None) == B.EINVAL
    B.check(B.lib.oases_op_gemm_tn_group(*args(601128256), ws.data_ptr(), ws.numel(), None))
    for i, (M, N) in enumerate(sizes):
        a, b = ab[i]
        ref = old[i].double() + a[:K].double().T @ b[:K].double()
        assert float((c[i].double() - ref).abs().max()) < K * 2.0 ** -24 * 4 * K ** 0.5
        single = old[i].clone()
        B.check(B.lib.oases_op_gemm_forced(601128256, B.GEMM_TN, B.EPI_F32, M, N, K, a.data_ptr(), a.shape[1], b.data_ptr(), b.shape[1], single.data_ptr(), N,
                                           None, None, 0, ws.data_ptr(), ws.numel(), None))
        assert torch.equal(single, c[i])


@pytest.mark.parametrize("op,epi,M,N,K,variants", [
    ("NN", "EPI_F32", 520, 328, 2112, (101256128, 101128256, 401064128, 301128256)), ("NT", "EPI_F32", 264, 520, 2048, (101256128, 101128256, 401064064, 301128256)),
    ("NN", "EPI_BIAS_BF16", 264, 264, 2048, (101256128, 301128256)), ("NT", "EPI_BF16", 136, 520, 2176, (101256128, 301128256)), ("NT", "EPI_DGELU", 520, 136, 2048, (101256128, 301128256)),
    ("TN", "EPI_F32", 520, 328, 2048, (101256128, 301128256)), ("TN", "EPI_F32", 264, 520, 2056, (101256128, 101128256, 401064064, 401064128, 501128128, 601128256)),
    ("TN", "EPI_F32", 136, 264, 1032, (101256128, 101128256, 401064128, 601128256)), ("TN", "EPI_F32", 136, 264, 1080, (101128256, 401064064, 601128256)),
    ("TN", "EPI_F32", 136, 264, 2112, (102128256, 402064128, 602128256)), ("TN", "EPI_F32", 264, 136, 4224, (104128256, 404064064, 604128256))])
def test_kernels_that_add_in_the_same_order(B, op, epi, M, N, K, variants):
    """Kernels between which the choice may change for speed alone give the same bits (wide rows of C and aux, odd multiples of eight)."""
    g = gen(M + N + K)
    a, b = randn(g, M, K).bfloat16(), (randn(g, K, N) * 0.05).bfloat16()
    ad, bd = padded(a if op != "TN" else a.t(), 0, 24), padded(b.t() if op == "NT" else b, 0, 8)
    opc, epi = getattr(B, "GEMM_" + op), getattr(B, epi)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    bias, aux = torch.randn(N, device="cuda"), torch.randn(M, N + 4, device="cuda").bfloat16()
    start, out = torch.randn(M, N + 4, device="cuda"), []
    for v in variants:
        c = start.clone() if epi == B.EPI_F32 else start.bfloat16()
        B.check(B.lib.oases_op_gemm_forced(v, opc, epi, M, N, K, ad.data_ptr(), ad.shape[1], bd.data_ptr(), bd.shape[1], c.data_ptr(), N + 4, bias.data_ptr(),
                                           aux.data_ptr(), N + 4, ws.data_ptr(), ws.numel(), None))
        out.append(c)
    for v, c in zip(variants[:-1], out):
        assert torch.equal(c, out[-1]), v
    assert torch.equal(out[-1][:, N:].float(), (start if epi == B.EPI_F32 else start.bfloat16())[:, N:].float()) and not torch.equal(out[-1].float(), start)
