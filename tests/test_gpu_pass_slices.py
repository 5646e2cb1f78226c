"""Products of a pass whose k slices the launch adds up itself: what a pass leaves in its workspace against the product of the operands
it leaves there, in 64 bits, twice in a workspace that starts as NaN with counters that are not zero."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# hidden, tp, tokens -> kernels with slices among the products of the pass (128x256 eight-wave tiles, small tiles, 128x128 tiles)
CASES = {(4096, 1, 136): {302128256}, (3072, 1, 264): {503128128, 402064128}, (2048, 1, 128): {404064064}, (4096, 1, 264): {304128256},
         (4096, 2, 400): {502128128}}


@pytest.mark.parametrize("h,tp,M", list(CASES))
def test_products_with_slices(h, tp, M):
    from paper_2305_16121_amd import binding as B
    cfg = dict(hidden=h, n_heads=h // 64, seq=M // 2, batch=2, tp=tp, n_sub=1, n_layers=1, causal=1, dropout_p=0.0)
    H = B.Handle(B.make_cfg(cfg, seed=1))
    hp, fp = h // tp, 4 * h // tp
    g = torch.Generator(device="cuda").manual_seed(h + M)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    W = dict(wqkv=n(h, 3 * hp) / h ** 0.5, wo=n(hp, h) / h ** 0.5, w1=n(h, fp) / h ** 0.5, w2=n(fp, h) / h ** 0.5)
    W = {k: v.bfloat16() for k, v in W.items()}
    W.update(bqkv=n(3 * hp), bo=n(h), b1=n(fp), b2=n(h), ln1_g=n(h), ln1_b=n(h), ln2_g=n(h), ln2_b=n(h))
    G = {k: torch.zeros(v.shape, device="cuda") for k, v in W.items()}
    x, dy, y, dx = n(M, h), n(M, h), torch.empty(M, h, device="cuda"), torch.empty(M, h, device="cuda")
    ws = torch.full((H.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")

    def tensor(name, cols, dtype):
        off, nb = H.tensor_span(name, 0)
        return ws[off:off + nb].view(dtype).view(M, cols)
    bf, f32 = torch.bfloat16, torch.float32
    # product, its operand and its weights; +bias where the epilogue has one
    products = [("NN", 2, tensor("qkv", 3 * hp, bf), tensor("u", h, bf), W["wqkv"], W["bqkv"]), ("NN", 0, tensor("z1", h, f32), tensor("attn", hp, bf), W["wo"], None),
                ("NN", 3, tensor("pre", fp, bf), tensor("v2", h, bf), W["w1"], W["b1"]), ("NN", 0, tensor("z2", h, f32), tensor("f", fp, bf), W["w2"], None),
                ("NT", 0, tensor("dv2", h, f32), tensor("dg", fp, bf), W["w1"], None), ("NT", 1, tensor("da", hp, bf), tensor("dz1", h, bf), W["wo"], None),
                ("NT", 0, tensor("du", h, f32), tensor("dqkv", 3 * hp, bf), W["wqkv"], None)]
    seen = {B.lib.oases_pass_gemm_variant({"NN": 0, "NT": 1}[op], epi, M, c.shape[1], a.shape[1], H.gemm_workspace_bytes) for op, epi, c, a, _, _ in products}
    assert CASES[(h, tp, M)] <= seen
    for _ in range(2):
        H.forward([W], x, y, ws)
        H.backward([W], x, dy, dx, [G], ws)
        torch.cuda.synchronize()
        for op, epi, c, a, w, bias in products:
            ref = a.double() @ (w.double() if op == "NN" else w.double().t().contiguous())
            if bias is not None:
                ref += bias.double()
            err = (c.double() - ref).abs()
            # fp32 sums of K products (K roundings at most of partial sums below the sum of their magnitudes), and half a bf16 ulp
            bound = a.shape[1] * 2.0 ** -24 * (a.double().abs() @ (w.double() if op == "NN" else w.double().t().contiguous()).abs())
            if c.dtype == bf:
                bound = bound + ref.abs() * 2.0 ** -8
            assert bool((err <= bound + 1e-30).all()), (op, epi, tuple(c.shape), float((err / (bound + 1e-30)).max()))
    H.close()


@pytest.mark.parametrize("M,h", [(200, 512), (72, 1024), (1032, 512), (2056, 256)])
def test_bias_gradients_that_come_with_the_weight_gradients(M, h):
    """Small-tile weight gradients add up the columns of their second operand on the way: the bias gradients of a pass against the column sums of
    the operands it leaves in its workspace, in 64 bits, accumulated into what was there; tokens that end inside a 64-wide tile of k."""
    from paper_2305_16121_amd import binding as B
    H = B.Handle(B.make_cfg(dict(hidden=h, n_heads=h // 64, seq=M // 8, batch=8, tp=1, n_sub=1, n_layers=1, causal=1, dropout_p=0.0), seed=1))
    g = torch.Generator(device="cuda").manual_seed(M)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    W = {k: (n(*s) / h ** 0.5).bfloat16() for k, s in dict(wqkv=(h, 3 * h), wo=(h, h), w1=(h, 4 * h), w2=(4 * h, h)).items()}
    W.update(bqkv=n(3 * h), bo=n(h), b1=n(4 * h), b2=n(h), ln1_g=n(h), ln1_b=n(h), ln2_g=n(h), ln2_b=n(h))
    G = {k: n(*v.shape) for k, v in W.items()}
    old = {k: G[k].clone() for k in ("b1", "bqkv")}
    x, y, dx = n(M, h), torch.empty(M, h, device="cuda"), torch.empty(M, h, device="cuda")
    ws = torch.full((H.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    H.forward([W], x, y, ws)
    H.backward([W], x, n(M, h), dx, [G], ws)
    torch.cuda.synchronize()
    for name, k, w in (("dg", "b1", 4 * h), ("dqkv", "bqkv", 3 * h)):
        off, nb = H.tensor_span(name, 0)
        t = ws[off:off + nb].view(torch.bfloat16).view(M, w).double()
        err = (G[k].double() - old[k].double() - t.sum(dim=0)).abs()
        # at most M / 16 + 64 roundings of partial sums below the sum of the magnitudes, and those of the old value and the result
        bound = (M / 16 + 64) * 2.0 ** -24 * t.abs().sum(dim=0) + 2.0 ** -23 * (old[k].abs() + G[k].abs()).double()
        assert bool((err <= bound).all()), (k, float((err / bound).max()))
    H.close()


# ..., kernel that leaves delta behind (0: none does, delta is the attention backward's own).  501128128 with 4608 and 1024 columns: the two
# launches of the attention backward; the others its single launch
@pytest.mark.parametrize("h,d,seq,batch,tp,causal,variant", [
    (512, 64, 72, 3, 1, 1, 401064064), (512, 128, 200, 1, 1, 1, 401064128), (1024, 64, 264, 2, 1, 1, 0), (2048, 128, 40, 5, 1, 1, 404064128),
    (2048, 64, 128, 1, 1, 1, 404064064), (4096, 64, 136, 2, 1, 1, 0),
    (4608, 64, 72, 1, 1, 1, 402064128),       # two heads a tile
    (5632, 64, 368, 1, 8, 1, 404064128),      # the same with an odd number of heads: the last tile holds one
    (10240, 64, 72, 1, 2, 1, 505128128),
    (1024, 128, 840, 3, 1, 0, 501128128),     # a last tile of 88 rows
    (4608, 128, 1376, 2, 4, 1, 501128128),
    (4608, 128, 200, 1, 1, 0, 503128128),     # a last tile of 72 rows
])
def test_delta_that_comes_with_the_gradient_of_the_attention_output(h, d, seq, batch, tp, causal, variant):
    """delta = rowsum(dO * O) per head, which small tiles that hold whole heads leave behind with dO (with and without k slices; last tiles of rows
    and of heads that are not whole, sequences that end inside a tile), against the arrays of the pass in 64 bits."""
    from paper_2305_16121_amd import binding as B
    M, hp, fp = seq * batch, h // tp, 4 * h // tp
    H = B.Handle(B.make_cfg(dict(hidden=h, n_heads=h // d, seq=seq, batch=batch, tp=tp, n_sub=1, n_layers=1, causal=causal, dropout_p=0.0), seed=1))
    assert H.pass_delta_variant == variant
    g = torch.Generator(device="cuda").manual_seed(M)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    W = {k: (n(*s) / h ** 0.5).bfloat16() for k, s in dict(wqkv=(h, 3 * hp), wo=(hp, h), w1=(h, fp), w2=(fp, h)).items()}
    W.update(bqkv=n(3 * hp), bo=n(h), b1=n(fp), b2=n(h), ln1_g=n(h), ln1_b=n(h), ln2_g=n(h), ln2_b=n(h))
    G = {k: torch.zeros(v.shape, device="cuda") for k, v in W.items()}
    x, y, dx = n(M, h), torch.empty(M, h, device="cuda"), torch.empty(M, h, device="cuda")
    ws = torch.full((H.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    H.forward([W], x, y, ws)
    H.backward([W], x, n(M, h), dx, [G], ws)
    torch.cuda.synchronize()

    def tensor(name, dtype):
        off, nb = H.tensor_span(name, 0)
        return ws[off:off + nb].view(dtype)
    products = (tensor("da", torch.bfloat16).double() * tensor("attn", torch.bfloat16).double()).view(batch, seq, hp // d, d)
    got = tensor("delta", torch.float32).double().view(batch, hp // d, seq)
    err = (got - products.sum(dim=3).transpose(1, 2)).abs()
    bound = d * 2.0 ** -24 * products.abs().sum(dim=3).transpose(1, 2)  # d roundings at most of partial sums below the sum of the magnitudes
    assert bool((err <= bound + 1e-30).all()), float((err / (bound + 1e-30)).max())
    H.close()


@pytest.mark.parametrize("d,seq,batch,p", [(64, 8, 1, 0.0), (64, 200, 2, 0.0), (64, 136, 1, 0.25), (128, 72, 3, 0.0), (128, 264, 1, 0.25)])
def test_gradients_turned_back_by_the_attention_backward(d, seq, batch, p):
    """A pass of few attention blocks stores dQ and dK turned back by the rotary embedding, with delta from the product that makes dO: against the
    attention backward and the inverse rotation as operators on the arrays that the pass leaves."""
    from paper_2305_16121_amd import binding as B
    h, heads, M = 8 * d, 8, seq * batch
    H = B.Handle(B.make_cfg(dict(arch="llama", hidden=h, n_heads=heads, ffn_hidden=2 * h, seq=seq, batch=batch, tp=1, n_sub=1, n_layers=1, causal=1,
                                 dropout_p=0.0, attn_dropout_p=p, rope_theta=10000.0), seed=7))
    g = torch.Generator(device="cuda").manual_seed(M + d)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    W = {k: (n(*s) / h ** 0.5).bfloat16() for k, s in dict(wqkv=(h, 3 * h), wo=(h, h), w1=(h, 4 * h), w2=(2 * h, h)).items()}
    W.update(ln1_g=n(h), ln2_g=n(h))
    G = {k: torch.zeros(v.shape, device="cuda") for k, v in W.items()}
    x, y, dx = n(M, h), torch.empty(M, h, device="cuda"), torch.empty(M, h, device="cuda")
    ws = torch.full((H.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    H.forward([W], x, y, ws)
    H.backward([W], x, n(M, h), dx, [G], ws)
    torch.cuda.synchronize()

    def at(name):
        off, nb = H.tensor_span(name, 0)
        return ws[off:off + nb]
    tab, delta = torch.empty(seq, d, device="cuda"), torch.empty(M * heads, device="cuda")
    ref = torch.empty(M, 3 * h, dtype=torch.bfloat16, device="cuda")
    B.check(B.lib.oases_op_rope_table(tab.data_ptr(), seq, d, 10000.0, None))
    B.check(B.lib.oases_op_attention_dropout_bwd(at("qkv").data_ptr(), at("attn").data_ptr(), at("da").data_ptr(), at("lse").data_ptr(), delta.data_ptr(),
                                                 ref.data_ptr(), batch, seq, heads, d, 1, 0, M, 7, 0, p, 0, heads, None))
    B.check(B.lib.oases_op_rope(ref.data_ptr(), 3 * h, M, 0, seq, heads, d, tab.data_ptr(), 1, None))
    torch.cuda.synchronize()
    got, ref = (t.view(torch.bfloat16).view(M, 3, heads, 2, d // 2).double() for t in (at("dqkv"), ref))
    # delta's sums run in another order: a value to be rotated may round to the neighbouring bf16, 2^-7 of it at most, which the rotation mixes into
    # both of a pair (at most sqrt 2 of the pair's length), and the result too; near zero, d + seq roundings of fp32 sums
    pair = (ref ** 2).sum(dim=3, keepdim=True).sqrt()
    bound = 2.0 ** -7 * (1.5 * pair + ref.abs()) + (d + seq) * 2.0 ** -24 * ref.abs().max() * 8
    assert bool(((got - ref).abs() <= bound).all()), float(((got - ref).abs() / bound).max())
    H.close()
