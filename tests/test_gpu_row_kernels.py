"""Row kernels at the widths where their split changes: a wave per row up to 1024 columns, 256 threads below 4096, 1024 threads
beyond (LayerNorm forward: 256 up to 4096), with whole and ragged chunks, and at few and odd numbers of rows."""
import pytest
import torch

from tests.util import rel_err

pytestmark = pytest.mark.gpu

WIDTHS = [8, 248, 256, 264, 520, 776, 1016, 1024, 1032, 2048, 2056, 3080, 4088, 4096, 4104, 8192, 8200, 12288, 16384]


def _rounds_to_bf16(got, ref):
    """Every element within half a unit of the last of bf16's eight bits (2^-8 of its value at most), plus the fp32 error."""
    rms = float(ref.pow(2).mean().sqrt())
    return bool(((got.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 4e-5 * rms).all())


def _ptr(t):
    return t.data_ptr() if t is not None else None


@pytest.mark.parametrize("h", WIDTHS)
@pytest.mark.parametrize("rows", [1, 7, 259, 1300])
def test_backward_row_kernels_against_fp64(h, rows):
    from paper_2305_16121_amd import binding as B
    if rows * h > 6_000_000:
        rows = 300
    gen = torch.Generator(device="cuda").manual_seed(h * 7 + rows)
    n = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    part, peer, dres, x = n(rows, h), n(rows, h), n(rows, h), n(rows, h) * 2 + 0.5
    gamma = n(h) * 0.1 + 1
    mu, rstd = x.mean(1), 1.0 / torch.sqrt(x.var(1, unbiased=False) + 1e-5)
    dxo = torch.full_like(x, float("nan"))
    dz = torch.full((rows, h), float("nan"), dtype=torch.bfloat16, device="cuda")
    sums = torch.ones(3, h, device="cuda")                    # accumulated into
    scratch = torch.full((3 * 1024 * h,), float("nan"), device="cuda")
    mask = torch.empty(rows, h, dtype=torch.uint8, device="cuda")
    seed, layer, site, row0, p = 5, 3, 1, 40, 0.25
    B.check(B.lib.oases_op_dropout_mask(_ptr(mask), seed, layer, site, row0, rows, h, p, None))
    B.check(B.lib.oases_op_layernorm_bwd(_ptr(part), _ptr(peer), _ptr(dres), _ptr(x), _ptr(mu), _ptr(rstd), _ptr(gamma), _ptr(dxo),
                                         _ptr(sums[0]), _ptr(sums[1]), _ptr(dz), _ptr(sums[2]), rows, h, seed, layer, site, row0, p,
                                         _ptr(scratch), None))
    torch.cuda.synchronize()
    d = torch.float64
    g, xh = part.to(d) + peer.to(d), (x.to(d) - mu.to(d)[:, None]) * rstd.to(d)[:, None]
    gg = g * gamma.to(d)
    ref = dres.to(d) + rstd.to(d)[:, None] * (gg - gg.mean(1, keepdim=True) - xh * (gg * xh).mean(1, keepdim=True))
    refz = torch.where(mask.bool(), ref / (1 - p), torch.zeros_like(ref))
    # fp32 arithmetic of sums of at most 16384 (row) and 1300 (column) terms: below 2e-5 of the root mean square per element
    assert rel_err(dxo, ref) < 2e-5
    assert _rounds_to_bf16(dz, refz)
    for got, want in ((sums[0], (g * xh).sum(0)), (sums[1], g.sum(0)), (sums[2], refz.sum(0))):
        assert rel_err(got, want + 1) < 2e-5
    # dropout backward of the same rows
    dz2 = torch.full_like(dz, float("nan"))
    db = torch.ones(h, device="cuda")
    B.check(B.lib.oases_op_dropout_bwd(_ptr(part), _ptr(dz2), _ptr(db), rows, h, seed, layer, site, row0, p, _ptr(scratch), None))
    torch.cuda.synchronize()
    refz = torch.where(mask.bool(), part.to(d) / (1 - p), torch.zeros_like(ref))
    assert _rounds_to_bf16(dz2, refz) and rel_err(db, refz.sum(0) + 1) < 2e-5


@pytest.mark.parametrize("h", WIDTHS)
@pytest.mark.parametrize("rows", [1, 37])
def test_forward_row_kernels_against_fp64(h, rows):
    from paper_2305_16121_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(h * 3 + rows)
    n = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    part, peer, xin, bias, gamma, beta = n(rows, h), n(rows, h), n(rows, h) * 2 + 3, n(h), n(h), n(h)
    xo, ln = torch.full_like(xin, float("nan")), torch.full((rows, h), float("nan"), dtype=torch.bfloat16, device="cuda")
    mu, rstd = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    mask = torch.empty(rows, h, dtype=torch.uint8, device="cuda")
    B.check(B.lib.oases_op_dropout_mask(_ptr(mask), 9, 1, 0, 8, rows, h, 0.25, None))
    B.check(B.lib.oases_op_bias_dropout_residual_ln(_ptr(part), _ptr(peer), _ptr(bias), _ptr(xin), _ptr(xo), _ptr(gamma), _ptr(beta),
                                                    _ptr(ln), _ptr(mu), _ptr(rstd), rows, h, 1e-5, 9, 1, 0, 8, 0.25, None))
    torch.cuda.synchronize()
    d = torch.float64
    z = part.to(d) + peer.to(d) + bias.to(d)
    ref = xin.to(d) + torch.where(mask.bool(), z / 0.75, torch.zeros_like(z))
    mean, var = ref.mean(1, keepdim=True), ref.var(1, unbiased=False, keepdim=True)
    want = (ref - mean) / torch.sqrt(var + 1e-5) * gamma.to(d) + beta.to(d)
    assert rel_err(xo, ref) < 2e-5 and rel_err(mu, mean[:, 0]) < 2e-5 and rel_err(rstd, 1 / torch.sqrt(var[:, 0] + 1e-5)) < 2e-5
    assert _rounds_to_bf16(ln, want)
    # the same row read back gives the same statistics and the same output, bit for bit
    ln2, mu2, rstd2 = torch.empty_like(ln), torch.empty_like(mu), torch.empty_like(rstd)
    B.check(B.lib.oases_op_layernorm_fwd(_ptr(xo), _ptr(gamma), _ptr(beta), _ptr(ln2), _ptr(mu2), _ptr(rstd2), rows, h, 1e-5, None))
    torch.cuda.synchronize()
    assert torch.equal(ln, ln2) and torch.equal(mu, mu2) and torch.equal(rstd, rstd2)


@pytest.mark.parametrize("cols", [8, 504, 512, 520, 1024, 1376])
@pytest.mark.parametrize("rows", [1, 5, 1021, 8200])
def test_column_sums_against_fp64(rows, cols):
    from paper_2305_16121_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    a = torch.randn(rows, cols + 16, generator=gen, device="cuda").to(torch.bfloat16)
    out = torch.ones(cols, device="cuda")
    scratch = torch.full((1024 * cols,), float("nan"), device="cuda")
    B.check(B.lib.oases_op_colsum_bf16(_ptr(a), cols + 16, rows, cols, _ptr(out), _ptr(scratch), None))
    torch.cuda.synchronize()
    assert rel_err(out, a[:, :cols].double().sum(0) + 1) < 2e-5


@pytest.mark.parametrize("h", [1024, 4096, 8192])
def test_rows_past_the_caches(h):
    """From 8 MiB of fp32 rows on the row kernels load and store past the caches: one row fewer, which goes the other way, gives the same rows bit for bit."""
    from paper_2305_16121_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(h)
    most = (8 << 20) // (4 * h)
    n = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    part, peer, dres, x = n(most, h), n(most, h), n(most, h), n(most, h)
    gamma, beta, bias = n(h), n(h), n(h)
    scratch = torch.empty(3 * 1024 * h, device="cuda")
    outs = []
    for rows in (most - 1, most):
        xo, dxo = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
        ln, dz, dz2 = (torch.full((most, h), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3))
        mu, rstd, sums = torch.empty(most, device="cuda"), torch.empty(most, device="cuda"), torch.zeros(4, h, device="cuda")
        B.check(B.lib.oases_op_bias_dropout_residual_ln(_ptr(part), _ptr(peer), _ptr(bias), _ptr(x), _ptr(xo), _ptr(gamma), _ptr(beta),
                                                        _ptr(ln), _ptr(mu), _ptr(rstd), rows, h, 1e-5, 9, 1, 0, 8, 0.25, None))
        B.check(B.lib.oases_op_layernorm_bwd(_ptr(part), _ptr(peer), _ptr(dres), _ptr(x), _ptr(mu), _ptr(rstd), _ptr(gamma), _ptr(dxo),
                                             _ptr(sums[0]), _ptr(sums[1]), _ptr(dz), _ptr(sums[2]), rows, h, 9, 1, 0, 8, 0.25, _ptr(scratch), None))
        B.check(B.lib.oases_op_dropout_bwd(_ptr(part), _ptr(dz2), _ptr(sums[3]), rows, h, 9, 1, 0, 8, 0.25, _ptr(scratch), None))
        torch.cuda.synchronize()
        assert bool(torch.isfinite(xo[:rows]).all()) and bool(torch.isnan(xo[rows:]).all()) and bool(torch.isnan(dxo[rows:]).all())
        outs.append([t[:most - 1] for t in (xo, ln, mu, rstd, dxo, dz, dz2)])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("rms", [False, True])
@pytest.mark.parametrize("h,rows", [(1024, 2048), (1024, 5121), (2056, 1027), (2056, 1285), (2056, 1799), (4096, 515)])
def test_streamed_rows_against_fp64(h, rows, rms):
    """Rows past the caches, LayerNorm and RMSNorm, with the column sums: workgroups that have one to three rows left in a loop that takes two (up to 1024
    columns) or four (below 4096) at a time."""
    from paper_2305_16121_amd import binding as B
    assert rows * h * 4 >= 8 << 20
    gen = torch.Generator(device="cuda").manual_seed(h + rows)
    n = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    d = torch.float64
    part, peer, dres, x, gamma = n(rows, h), n(rows, h), n(rows, h), n(rows, h), n(h) * 0.1 + 1
    beta, bias = (torch.zeros(h, device="cuda"),) * 2 if rms else (n(h), n(h))
    mask, scratch = torch.empty(rows, h, dtype=torch.uint8, device="cuda"), torch.full((3 * 1024 * h,), float("nan"), device="cuda")
    drop = (9, 1, 0, 8, 0.25)                    # seed, layer, site, first row, rate
    B.check(B.lib.oases_op_dropout_mask(_ptr(mask), *drop[:4], rows, h, 0.25, None))
    keep = lambda t: torch.where(mask.bool(), t / 0.75, torch.zeros_like(t))
    # forward
    xo, ln = torch.full_like(x, float("nan")), torch.full((rows, h), float("nan"), dtype=torch.bfloat16, device="cuda")
    mu, rstd = torch.zeros(rows, device="cuda"), torch.empty(rows, device="cuda")
    if rms:
        B.check(B.lib.oases_op_dropout_residual_rmsnorm(_ptr(part), _ptr(peer), _ptr(x), _ptr(xo), _ptr(gamma), _ptr(ln), _ptr(rstd), rows, h, 1e-5, *drop, None))
    else:
        B.check(B.lib.oases_op_bias_dropout_residual_ln(_ptr(part), _ptr(peer), _ptr(bias), _ptr(x), _ptr(xo), _ptr(gamma), _ptr(beta), _ptr(ln), _ptr(mu), _ptr(rstd),
                                                        rows, h, 1e-5, *drop, None))
    torch.cuda.synchronize()
    ref = x.to(d) + keep(part.to(d) + peer.to(d) + bias.to(d))
    mean = torch.zeros(rows, 1, dtype=d, device="cuda") if rms else ref.mean(1, keepdim=True)
    r = 1 / torch.sqrt(((ref - mean) ** 2).mean(1, keepdim=True) + 1e-5)
    assert rel_err(xo, ref) < 2e-5 and rel_err(rstd, r[:, 0]) < 2e-5 and (rms or rel_err(mu, mean[:, 0]) < 2e-5)
    assert _rounds_to_bf16(ln, (ref - mean) * r * gamma.to(d) + beta.to(d))
    # backward of the rows x with these statistics
    dxo, dz, sums = torch.full_like(x, float("nan")), torch.full_like(ln, float("nan")), torch.ones(4, h, device="cuda")
    if rms:
        B.check(B.lib.oases_op_rmsnorm_bwd(_ptr(part), _ptr(peer), _ptr(dres), _ptr(x), _ptr(rstd), _ptr(gamma), _ptr(dxo), _ptr(sums[0]), _ptr(dz), rows, h, *drop,
                                           _ptr(scratch), None))
    else:
        B.check(B.lib.oases_op_layernorm_bwd(_ptr(part), _ptr(peer), _ptr(dres), _ptr(x), _ptr(mu), _ptr(rstd), _ptr(gamma), _ptr(dxo), _ptr(sums[0]), _ptr(sums[1]),
                                             _ptr(dz), _ptr(sums[2]), rows, h, *drop, _ptr(scratch), None))
    dz2 = torch.full_like(ln, float("nan"))
    B.check(B.lib.oases_op_dropout_bwd(_ptr(part), _ptr(dz2), _ptr(sums[3]), rows, h, *drop, _ptr(scratch), None))
    torch.cuda.synchronize()
    g, xh = part.to(d) + peer.to(d), (x.to(d) - mu.to(d)[:, None]) * rstd.to(d)[:, None]
    gg = g * gamma.to(d)
    ref = dres.to(d) + rstd.to(d)[:, None] * (gg - (0 if rms else gg.mean(1, keepdim=True)) - xh * (gg * xh).mean(1, keepdim=True))
    assert rel_err(dxo, ref) < 2e-5 and _rounds_to_bf16(dz, keep(ref)) and _rounds_to_bf16(dz2, keep(part.to(d)))
    want = [(g * xh).sum(0), g.sum(0), keep(ref).sum(0), keep(part.to(d)).sum(0)]
    for i in (0, 3) if rms else range(4):
        assert rel_err(sums[i], want[i] + 1) < 2e-5, i


@pytest.mark.parametrize("h,rows", [(1024, 2048), (1024, 2040), (2048, 1288)])
def test_post_layernorm_rows_of_a_pass_against_fp64(h, rows):
    """The post-LayerNorm forms, which only passes use (2040 rows of 1024: below the 8 MiB from which rows go past the caches): what a pass leaves in its
    workspace against the definition on the arrays that it read."""
    from paper_2305_16121_amd import binding as B
    H = B.Handle(B.make_cfg(dict(arch="bert", hidden=h, n_heads=h // 64, seq=8, batch=rows // 8, tp=1, n_sub=1, n_layers=1, causal=0, dropout_p=0.25), seed=9))
    gen = torch.Generator(device="cuda").manual_seed(h + rows)
    n = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    W = {k: (n(*s) / h ** 0.5).bfloat16() for k, s in dict(wqkv=(h, 3 * h), wo=(h, h), w1=(h, 4 * h), w2=(4 * h, h)).items()}
    W.update(bqkv=n(3 * h), bo=n(h), b1=n(4 * h), b2=n(h), ln1_g=n(h), ln1_b=n(h), ln2_g=n(h), ln2_b=n(h))
    G = {k: torch.zeros(v.shape, device="cuda") for k, v in W.items()}
    x, dy, y, dx = n(rows, h), n(rows, h), torch.empty(rows, h, device="cuda"), torch.empty(rows, h, device="cuda")
    ws = torch.full((H.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    H.forward([W], x, y, ws)
    H.backward([W], x, dy, dx, [G], ws)
    torch.cuda.synchronize()
    d = torch.float64

    def at(name, dtype=torch.float32):
        off, nb = H.tensor_span(name, 0)
        return ws[off:off + nb].view(dtype).view(rows, -1).to(d)
    keep = []
    for site in (0, 1):
        mask = torch.empty(rows, h, dtype=torch.uint8, device="cuda")
        B.check(B.lib.oases_op_dropout_mask(_ptr(mask), 9, 0, site, 0, rows, h, 0.25, None))
        keep.append(lambda t, m=mask.bool(): torch.where(m, t / 0.75, torch.zeros_like(t)))
    # forward: the sums in front of the two LayerNorms, and their rows in fp32 and bf16
    for xin, z, bias, s, site, ln, out in ((x.to(d), "z1", "bo", "s1", 0, "ln1", at("x1")), (at("x1"), "z2", "b2", "s2", 1, "ln2", y.to(d))):
        ref = xin + keep[site](at(z) + W[bias].to(d))
        assert rel_err(at(s), ref) < 2e-5, s
        s = at(s)
        want = (s - s.mean(1, keepdim=True)) / torch.sqrt(s.var(1, unbiased=False, keepdim=True) + 1e-5) * W[ln + "_g"].to(d) + W[ln + "_b"].to(d)
        assert rel_err(out, want) < 2e-5, ln
    assert _rounds_to_bf16(at("v2", torch.bfloat16), at("x1"))
    # backward: LN2 and the dropout of the FFN branch, then LN1 and that of the attention branch
    for g, s, ln, m, out, dz, db, site in ((dy.to(d), "s2", "ln2", "2", "ds2", "dz2", "b2", 1), (at("dv2") + at("ds2"), "s1", "ln1", "1", "dx1", "dz1", "bo", 0)):
        xh = (at(s) - at("mu" + m)) * at("rstd" + m)
        gg = g * W[ln + "_g"].to(d)
        ref = at("rstd" + m) * (gg - gg.mean(1, keepdim=True) - xh * (gg * xh).mean(1, keepdim=True))
        assert rel_err(at(out), ref) < 2e-5 and _rounds_to_bf16(at(dz, torch.bfloat16), keep[site](ref)), ln
        for got, want in ((G[ln + "_g"], (g * xh).sum(0)), (G[ln + "_b"], g.sum(0)), (G[db], keep[site](ref).sum(0))):
            assert rel_err(got, want) < 2e-5, (ln, db)
    H.close()
