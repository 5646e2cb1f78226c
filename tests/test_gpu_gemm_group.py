"""Two weight gradients in one launch (oases_op_gemm_tn_group): every kernel and slice count it has, whole and ragged tiles,
against a matrix product in 64 bits and, where a single launch has the same kernel and slices, against that bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu

WS = 4096 + 64 * 8 * 128 * 256 * 4


@pytest.fixture(scope="module")
def B():
    from paper_2305_16121_amd import binding
    return binding


def problem(K, M, N, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn(K, M + 8, generator=g, device="cuda").bfloat16()
    b = torch.randn(K, N + 16, generator=g, device="cuda").bfloat16()
    c = torch.randn(M, N + 4, generator=g, device="cuda")
    return a, b, c


def call(B, variant, K, p, q, ws, nbytes=None):
    args = [variant, K]
    for (a, b, c), M, N in (p, q):
        args += [M, N, a.data_ptr(), a.shape[1], b.data_ptr(), b.shape[1], c.data_ptr(), c.shape[1]]
    return B.lib.oases_op_gemm_tn_group(*args, ws.data_ptr() if ws is not None else None, (ws.numel() if nbytes is None else nbytes) if ws is not None else 0, None)


@pytest.mark.parametrize("variant", [0, 301128256, 302128256, 304128256, 308128256, 401064064, 401064128])
@pytest.mark.parametrize("K,M0,N0,M1,N1", [(1024, 256, 512, 128, 256), (1024, 136, 264, 8, 1000), (704, 120, 256, 384, 8), (512, 128, 8, 8, 256)])
def test_group_against_the_product_in_64_bits(B, variant, K, M0, N0, M1, N1):
    ws = torch.full((WS,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN partial sums, counters that are not zero
    p, q = problem(K, M0, N0, 1), problem(K, M1, N1, 2)
    before = [x[2].clone() for x in (p, q)]
    S = variant // 1000000 % 100
    rc = call(B, variant, K, (p, M0, N0), (q, M1, N1), ws)
    if S == 8 and K == 704:      # eleven stages: the last two of eight slices would have none
        assert rc == B.EINVAL
        return
    B.check(rc)
    torch.cuda.synchronize()
    assert bool((ws[:4096].view(torch.int32) == 0).all())             # every counter is back at zero
    for (a, b, c), old, M, N in ((p, before[0], M0, N0), (q, before[1], M1, N1)):
        ref = old[:, :N].double() + a[:, :M].double().T @ b[:, :N].double()
        # fp32 sums of K products of bf16 numbers of unit variance: K roundings of partial sums of size sqrt(K) at most
        assert float((c[:, :N].double() - ref).abs().max()) < K * 2.0 ** -24 * 4 * K ** 0.5
        assert torch.equal(c[:, N:], old[:, N:])                      # nothing beyond the columns
        single = old.clone()
        if variant and K % (64 * S) == 0 and variant != 308128256:
            B.check(B.lib.oases_op_gemm_forced(variant, B.GEMM_TN, B.EPI_F32, M, N, K, a.data_ptr(), a.shape[1], b.data_ptr(), b.shape[1],
                                               single.data_ptr(), single.shape[1], None, None, 0, ws.data_ptr(), ws.numel(), None))
            assert torch.equal(single, c)


def test_group_refusals(B):
    K, M, N = 256, 128, 256
    p, q, ws = problem(K, M, N, 1), problem(K, M, N, 2), torch.empty(WS, dtype=torch.uint8, device="cuda")
    rc = lambda v, w=ws, n=None: call(B, v, K, (p, M, N), (q, M, N), w, n)
    assert rc(302128256) == B.OK and rc(0, None) == B.OK
    assert rc(302128256, None) == B.EINVAL
    assert rc(302128256, ws, 4096 + 2 * 2 * 128 * 256 * 4 - 4) == B.EINVAL
    assert rc(303128256) == B.EINVAL and rc(308128256) == B.EINVAL and rc(402064064) == B.EINVAL and rc(301256256) == B.EINVAL
    assert rc(-1) == B.EINVAL
