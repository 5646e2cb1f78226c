"""The attention kernels on both sides of every rule that picks their block shape: one or two row groups per workgroup, one
launch or two for the backward, shared or wave-private tiles; sequences that end inside a tile, and scores whose running
maximum moves in large and in small steps."""
import math

import pytest
import torch

from tests.util import rms_err, bf16_round, assert_bf16_close, dev, randn

pytestmark = pytest.mark.gpu

#        batch, seq, heads, d, causal, p            64-row blocks / 32-row blocks
CASES = [(32, 72, 8, 64, 1, 0.0),                   # 512 / 768: two groups, the second block holds eight rows
         (32, 72, 8, 128, 0, 0.0),
         (8, 200, 16, 128, 1, 0.0),                 # 512 / 896
         (8, 200, 16, 64, 1, 0.2),
         (8, 200, 16, 128, 0, 0.2),
         (16, 96, 8, 128, 1, 0.3),                  # 256 / 384, short: two groups
         (2, 520, 8, 64, 1, 0.0),                   # 144 / 272: one group, two launches
         (2, 520, 8, 64, 0, 0.1),
         (2, 520, 8, 128, 1, 0.0),                  # wave-private dQ and dK/dV
         (2, 520, 8, 128, 0, 0.25),
         (2, 264, 10, 64, 1, 0.1),                  # 100 / 180: dropout, two launches
         (2, 264, 6, 64, 1, 0.1),                   # 60 / 108: dropout, one launch
         (2, 264, 6, 128, 1, 0.1),                  # forward: one group, dropout
         (16, 72, 10, 64, 1, 0.0),                  # 320 of two blocks a sequence: forward workgroups from 256 on take theirs in the other order
         (4, 512, 10, 64, 1, 0.0)]                  # 320 of eight


@pytest.mark.parametrize("batch,seq,heads,d,causal,p", CASES)
@pytest.mark.parametrize("ramp", [0.0, 6.0])
def test_attention_blocks(batch, seq, heads, d, causal, p, ramp):
    from oracle import layer_oracle as lo
    from paper_2305_16121_amd import binding as B
    g = torch.Generator().manual_seed(seq + d)
    M, hp = batch * seq, heads * d
    qkv, dout = randn(g, M, 3 * hp), randn(g, M, hp)
    if ramp:   # keys that grow along the sequence: the running maximum rises in every tile, by little and by much
        qkv[:, hp:2 * hp] *= (0.2 + ramp * torch.arange(M, dtype=torch.float64).remainder(seq) / seq)[:, None]
        qkv[:, :hp] *= 0.5
    qkv, dout = bf16_round(qkv), bf16_round(dout)
    q, k, v = qkv[:, :hp], qkv[:, hp:2 * hp], qkv[:, 2 * hp:]
    seed, layer, head0, heads_total = 77, 1, 2, heads + 3
    drop = lo.attention_dropout_factor(seed, layer, batch, seq, heads_total, head0, heads, p) if p else 1.0
    A, P = lo.attention_fwd(q, k, v, batch, seq, heads, d, causal, drop=drop if p else None)
    qd, dod = dev(qkv, torch.bfloat16), dev(dout, torch.bfloat16)
    nan = float("nan")
    out = torch.full((M, hp), nan, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((batch * heads * seq,), nan, device="cuda")
    delta, dqkv = torch.full_like(lse, nan), torch.full((M, 3 * hp), nan, dtype=torch.bfloat16, device="cuda")
    B.check(B.lib.oases_op_attention_dropout_fwd(qd.data_ptr(), out.data_ptr(), lse.data_ptr(), batch, seq, heads, d, causal, 0, M, seed, layer, p,
                                                 head0, heads_total, None))
    B.check(B.lib.oases_op_attention_dropout_bwd(qd.data_ptr(), out.data_ptr(), dod.data_ptr(), lse.data_ptr(), delta.data_ptr(), dqkv.data_ptr(),
                                                 batch, seq, heads, d, causal, 0, M, seed, layer, p, head0, heads_total, None))
    torch.cuda.synchronize()
    scale = 256.0 / (256.0 - round(256 * p))
    # every weight P D is rounded to bf16 in front of P V: half a unit of the last place, 2^-8 of it at most; the weights of a row
    # sum to at most about `scale`
    assert_bf16_close(out.float(), A, 0.0, 2.0 ** -8 * scale * float(v.abs().max()), "attention forward")
    H, U = (lambda t: lo._heads(t, batch, seq, heads, d)), (lambda t: lo._unheads(t, batch, seq, heads, d))
    S = (H(q) @ H(k).transpose(2, 3)) / math.sqrt(d)
    if causal:
        i = torch.arange(seq)
        S = S.masked_fill(i[None, :] > i[:, None], float("-inf"))
    assert float((lse.cpu().double().reshape(batch, heads, seq) - torch.logsumexp(S, dim=3)).abs().max()) < 2e-3
    # the backward with the kernel's storage roundings written out: delta from the bf16 output, P and dS rounded to bf16 where they
    # enter a matrix product.  What remains is the final rounding and roundings of P / dS that fall the other way, each of which
    # moves one term of a sum by at most 2^-8 of it: rare, so small in the mean, and bounded per element by one flip of the
    # largest term (scores of up to s give the exponent 2^-24 s of relative error in fp32, far below that)
    dl = (H(dout) * H(out.float().cpu().double())).sum(dim=3, keepdim=True)
    assert rms_err(delta.reshape(batch, heads, seq), dl[..., 0]) < 1e-5
    dS = P * ((H(dout) @ H(v).transpose(2, 3)) * drop - dl)
    ref = dict(dq=U(bf16_round(dS) @ H(k)) / math.sqrt(d), dk=U(bf16_round(dS).transpose(2, 3) @ H(q)) / math.sqrt(d),
               dv=U(bf16_round(P * drop).transpose(2, 3) @ H(dout)))
    flip = 2.0 ** -8 * float(dS.abs().max()) / math.sqrt(d)
    flips = dict(dq=flip * float(k.abs().max()), dk=flip * float(q.abs().max()), dv=2.0 ** -8 * scale * float(dout.abs().max()))
    got = dqkv.float().cpu().double()
    for n, (name, r) in enumerate(ref.items()):
        part = got[:, n * hp:(n + 1) * hp]
        assert rms_err(part, r) < 3e-3, name
        assert_bf16_close(part, r, 3e-3, flips[name], name)


@pytest.mark.parametrize("batch,seq,heads,d,causal,parts", [(4, 1024, 8, 64, 1, 2), (8, 512, 8, 128, 0, 2), (1, 1024, 4, 128, 1, 4), (1, 1000, 4, 64, 0, 4)])
def test_probabilities_are_rounded_relative_to_the_largest_score(batch, seq, heads, d, causal, parts):
    """The output's error is that of the definition with its probabilities rounded to bf16 relative to the largest score so far, tile
    by tile of 32 keys dealt out to `parts` partial sums, and no more: over 2^19 and more elements the ratio of the two
    repeats to a per cent (a reference that lags behind by up to 2^6 makes it 1.08 to 1.15)."""
    from paper_2305_16121_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(seq + d)
    M, hp = batch * seq, heads * d
    qkv = (2.0 * torch.randn(M, 3 * hp, generator=g, device="cuda")).bfloat16()
    q, k, v = (t.reshape(batch, seq, heads, d).transpose(1, 2).double() for t in qkv.split(hp, dim=1))
    S = (q @ k.transpose(2, 3).contiguous()) * (math.log2(math.e) / math.sqrt(d))
    if causal:
        S = S.masked_fill(torch.ones(seq, seq, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    exact = torch.softmax(S * math.log(2.0), dim=3) @ v
    tiles = torch.nn.functional.pad(S, (0, -seq % 32), value=float("-inf")).unflatten(3, (-1, 32))
    top = tiles.amax(dim=4)
    for p in range(parts):
        top[..., p::parts] = top[..., p::parts].cummax(dim=3).values
    top = top.clamp_min(-1e30)
    P = torch.exp2(tiles - top[..., None])
    w = torch.exp2(top - top.amax(dim=3, keepdim=True))[..., None]
    P8 = P.bfloat16().double()
    model = ((P8 * w).flatten(3)[..., :seq] @ v) / (P * w).flatten(3).sum(dim=3, keepdim=True)
    out = torch.full((M, hp), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty(batch * heads * seq, device="cuda")
    B.check(B.lib.oases_op_attention_fwd(qkv.data_ptr(), out.data_ptr(), lse.data_ptr(), batch, seq, heads, d, causal, 0, M, None))
    got = out.double().reshape(batch, seq, heads, d).transpose(1, 2)
    e, bound = rms_err(got, exact), rms_err(model.bfloat16(), exact)
    print(f"error {e:.6f}, of the definition {bound:.6f}, ratio {e / bound:.4f}")
    assert e < 1.03 * bound


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [2, 64])          # wave-private tiles in one launch; two groups per workgroup
@pytest.mark.parametrize("row0,rows,p", [(0, 520, 0.0), (520, 504, 0.0), (8, 1016, 0.1), (6, 514, 0.1), (513, 398, 0.2), (3, 5, 0.1)])
def test_row_range_agrees_with_the_whole_sequence(d, heads, row0, rows, p):
    """A row range of one sequence, with blocks that start at the range (also where that is no multiple of the mask's four) and end
    inside a tile, gives the rows of the whole call up to the roundings of another block split."""
    from paper_2305_16121_amd import binding as B
    seq = 1024
    hp = heads * d
    g = torch.Generator(device="cuda").manual_seed(d + row0)
    qkv = torch.randn(seq, 3 * hp, generator=g, device="cuda").bfloat16()
    dout = torch.randn(seq, hp, generator=g, device="cuda").bfloat16()

    def run(r0, n, base=None):
        out = base[0].clone() if base else torch.zeros(seq, hp, dtype=torch.bfloat16, device="cuda")
        lse = base[1].clone() if base else torch.zeros(heads * seq, device="cuda")
        delta, dqkv = torch.full_like(lse, float("nan")), torch.full_like(qkv, 7.0)
        B.check(B.lib.oases_op_attention_dropout_fwd(qkv.data_ptr(), out.data_ptr(), lse.data_ptr(), 1, seq, heads, d, 1, r0, n, 5, 1, p, 0, heads, None))
        B.check(B.lib.oases_op_attention_dropout_bwd(qkv.data_ptr(), out.data_ptr(), dout.data_ptr(), lse.data_ptr(), delta.data_ptr(),
                                                     dqkv.data_ptr(), 1, seq, heads, d, 1, r0, n, 5, 1, p, 0, heads, None))
        torch.cuda.synchronize()
        return out, lse, dqkv

    whole = run(0, seq)
    part = run(row0, rows, whole)
    rs = slice(row0, row0 + rows)
    assert rms_err(part[0][rs], whole[0][rs]) < 4e-3 and rms_err(part[1], whole[1]) < 1e-5
    for n in range(3):
        assert rms_err(part[2][rs, n * hp:(n + 1) * hp], whole[2][rs, n * hp:(n + 1) * hp]) < 6e-3
    outside = torch.cat([part[2][:row0], part[2][row0 + rows:]])
    assert bool((outside == 7.0).all())                        # no row outside the range is written
