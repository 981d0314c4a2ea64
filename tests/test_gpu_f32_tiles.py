"""fp32 products on the matrix cores and attention with a wavefront per query: the small shapes against float64 and against the
large ones, bit for bit, at the edges of tiles, k-tiles and query chunks."""
import pytest
import torch

import paper_2511_18191_amd as tsd
from synth import ModelCfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,big", [
    (1, 64, 16, 9000), (17, 48, 64, 9000), (40, 64, 256, 9000), (33, 132, 104, 4200),   # K below, at, over and off the k-tiles
    (16, 192, 32, 4200), (15, 256, 128, 4200), (64, 8, 1032, 9000),
])
def test_fp32_products_of_few_and_of_many_rows(M, N, K, big):
    g = torch.Generator().manual_seed(M + N + K)
    A = torch.randn(big, K, generator=g).cuda()
    W = (torch.randn(N, K, generator=g) * 0.05).cuda()
    a, w = A[:M].cpu().double(), W.cpu().double()
    for variant in (0, 1, 2):
        few, many = (torch.full((m, N), 0.5, device="cuda") for m in (M, big))
        tsd.bench_gemm(A[:M].contiguous(), W, out=few, variant=variant)
        tsd.bench_gemm(A, W, out=many, variant=variant)
        torch.cuda.synchronize()
        assert torch.equal(few, many[:M]), variant
        ref, size = a @ w.T, a.abs() @ w.abs().T
        if variant == 1:
            scale = torch.rsqrt((a * a).mean(-1, keepdim=True) + 1e-6)
            ref, size = ref * scale, size * scale
        if variant == 2:
            ref, size = ref + 0.5, size + 0.5
        # a chain of K fused multiply-adds rounds K times; the row scale's own sum and the result's last steps the same again
        assert ((few.cpu().double() - ref).abs() <= (2 * K + 8) * 2.0 ** -24 * size).all(), variant


@pytest.mark.parametrize("D,heads,N,K", [(64, 4, 20, 4), (64, 2, 9, 1), (128, 2, 8, 7), (64, 4, 33, 8)])
def test_fp32_series_alone_and_among_many_same_bits(D, heads, N, K):
    """Three series: 16-row tiles and a wavefront per query.  The same ones among many: 64-row tiles, a wavefront per head."""
    P, T = 16, 5
    many = 2100 // heads
    m = ModelCfg(2, D, heads, 4 * D)
    g = torch.Generator().manual_seed(D + heads + N)
    n = P * D + 2 * (2 * D + 4 * D * D + 8 * D * D) + D + D * P
    w = torch.randn(n, generator=g) * 0.05
    series = torch.randn(many, N * P, generator=g)
    res = []
    for B in (3, many):
        sess = tsd.Session(tsd.make_config(m, m, P, K, B, N + T + K, "fp32", 1.0, seed=3))
        for which in (tsd.TSD_TARGET, tsd.TSD_DRAFT):
            sess.load_weights(which, w.cuda())
        sess.prefill(series[:B].cuda(), N, T * P)
        sess.round()
        io = sess.get_round_io()
        res.append({k: io[k][:3].cpu() for k in ("X", "mu_p")})
        sess.run_rounds()
        res[-1]["forecast"] = sess.get_forecast()[:3].cpu()
        sess.close()
    for k in res[0]:
        assert torch.isfinite(res[0][k]).all() and torch.equal(res[0][k], res[1][k]), k
