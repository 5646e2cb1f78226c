"""Sums that ride on the small-tile kernels run in one fixed order of fp32 additions, whatever shape of MFMA the kernel multiplies with: bias gradients
(column sums of a weight gradient's second operand) and delta = rowsum(dO * O), each against the same additions, in that order, on the arrays that a
pass leaves: delta, which is rounded into dQ and dK, so that another order is another gradient, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def one_pass(cfg):
    from paper_2305_16121_amd import binding as B
    H = B.Handle(B.make_cfg(cfg, seed=1))
    h, M = cfg["hidden"], cfg["seq"] * cfg["batch"]
    hp, fp = h // cfg["tp"], 4 * h // cfg["tp"]
    g = torch.Generator(device="cuda").manual_seed(M + h)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    W = {k: (n(*s) / h ** 0.5).bfloat16() for k, s in dict(wqkv=(h, 3 * hp), wo=(hp, h), w1=(h, fp), w2=(fp, h)).items()}
    W.update(bqkv=n(3 * hp), bo=n(h), b1=n(fp), b2=n(h), ln1_g=n(h), ln1_b=n(h), ln2_g=n(h), ln2_b=n(h))
    G = {k: torch.zeros(v.shape, device="cuda") for k, v in W.items()}
    x, dy, y, dx = n(M, h), n(M, h), torch.empty(M, h, device="cuda"), torch.empty(M, h, device="cuda")
    ws = torch.full((H.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    H.forward([W], x, y, ws)
    H.backward([W], x, dy, dx, [G], ws)
    torch.cuda.synchronize()

    def tensor(name, dtype):
        off, nb = H.tensor_span(name, 0)
        return ws[off:off + nb].view(dtype)
    return H, tensor, G


def in_order(terms):
    """terms[0] + terms[1] + ... one after the other."""
    s = terms[0]
    for t in terms[1:]:
        s = s + t
    return s


def column_sums(t):
    """[K, N] in fp32, 64 k to a tile and zeros behind K.  A wave has 32 k of a tile: its lanes hold eight k each and add up those of every second eight; a
    partial sum is eight tiles."""
    K, N = t.shape
    nk = -(-K // 64)
    t = torch.cat([t, t.new_zeros(nk * 64 - K, N)]).view(nk, 2, 2, 2, 4, 2, N)  # tile, wave, 16 k, b, pair, of a pair
    eight = in_order([t[:, :, :, :, i // 2, i % 2] for i in range(8)])
    step = eight[:, :, 0] + eight[:, :, 1]                                        # tile, wave, b, N
    total, part = torch.zeros_like(step[0]), torch.zeros_like(step[0])
    for kt in range(nk):
        part = part + step[kt]
        if kt % 8 == 7:
            total, part = total + part, torch.zeros_like(part)
    total = total + part
    both = total[0] + total[1]                                                    # b, N
    return both[0] + both[1]


@pytest.mark.parametrize("M,h", [(200, 512), (72, 1024), (1032, 512), (2056, 256)])
def test_bias_gradients(M, h):
    """v_dot2_f32_bf16, which adds two values to a sum, does not round as two additions do: up to 2.5 % of the columns come out another way (the key
    columns of bqkv, whose sums cancel).  With one other step of the order, k rows that are 16 apart in chains of their own, it is 9 to 25 %."""
    H, tensor, G = one_pass(dict(hidden=h, n_heads=h // 64, seq=M // 8, batch=8, tp=1, n_sub=1, n_layers=1, causal=1, dropout_p=0.0))
    for name, k, w in (("dg", "b1", 4 * h), ("dqkv", "bqkv", 3 * h)):
        other = float((G[k] != column_sums(tensor(name, torch.bfloat16).view(M, w).float())).float().mean())
        assert other < 0.05, (k, other)
    H.close()


@pytest.mark.parametrize("h,d,seq,batch,tp,variant", [(512, 64, 72, 3, 1, 401064064), (512, 128, 200, 1, 1, 401064128), (2048, 128, 40, 5, 1, 404064128),
                                                       (2048, 64, 128, 1, 1, 404064064), (4608, 64, 72, 1, 1, 402064128), (5632, 64, 368, 1, 8, 404064128),
                                                       (10240, 64, 72, 1, 2, 505128128), (4608, 128, 1376, 2, 4, 501128128)])
def test_delta(h, d, seq, batch, tp, variant):
    """Per wave and 32 columns four chains of columns 16 H + 8 q + 4 b + e (H, b = 0, 1) that run through q, the wave's parts of 32 and e; then both b, both H,
    both waves of a head."""
    H, tensor, _ = one_pass(dict(hidden=h, n_heads=h // d, seq=seq, batch=batch, tp=tp, n_sub=1, n_layers=1, causal=1, dropout_p=0.0))
    assert H.pass_delta_variant == variant
    heads, bn = h // tp // d, variant % 1000
    waves = 2 if d == bn else 1
    p = (tensor("da", torch.bfloat16).float() * tensor("attn", torch.bfloat16).float()).view(batch, seq, heads, waves, d // waves // 32, 2, 2, 2, 4)  # .., part, H, q, b, e
    s = in_order([p[..., j, :, q, :, e] for q in range(2) for j in range(p.shape[4]) for e in range(4)])  # ..., wave, H, b
    s = s[..., 0] + s[..., 1]
    s = s[..., 0] + s[..., 1]
    s = in_order(list(s.unbind(-1)))
    assert torch.equal(tensor("delta", torch.float32).view(batch, heads, seq), s.transpose(1, 2))
    H.close()
