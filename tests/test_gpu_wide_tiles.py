"""The wide direct-to-LDS tiles (128 x 64 up to 256 x 256) against the register-staged kernels, bit for bit, and against float64, at the
edges of their shapes: shortest contractions, last tiles of a few rows, every rotary layout."""
import pytest
import torch

import paper_2511_18191_amd as tsd
from synth import ModelCfg

pytestmark = pytest.mark.gpu
QKV, RESID, GELU = 1, 3, 4  # TSD_K_QKV, TSD_K_RESID, TSD_K_GELU
# rows, columns, k, variant of tsd_bench_gemm, the tile they take (tests/test_gemm_tiles.py holds the rule to it)
PRODUCTS = [
    (6529, 2048, 192, 3, 257), (13057, 1024, 256, 3, 257), (6401, 2048, 192, 3, 257),   # 256 x 256: three k-tiles, a last tile of one row
    (321, 4096, 192, 3, 127), (321, 4096, 256, 3, 127), (1281, 4160, 320, 3, 127),      # 128 x 64: two stages, three, columns of no 128-multiple
    (6401, 1152, 192, 3, 128), (4097, 3200, 512, 3, 128), (4480, 1024, 2048, 1, 128),   # 128 x 128 behind the norm, long too
    (4500, 768, 512, 2, 128), (2817, 1280, 1088, 0, 128),                               # 128 x 128 with three stages, four runs of k-tiles
    (4500, 768, 256, 2, 64),                                                            # ... too short for them
    (6529, 1024, 512, 2, 128), (16300, 384, 192, 0, 128),                               # ... with two
    (4400, 1024, 2112, 2, 256), (8999, 512, 2048, 0, 256),                              # 256 x 128: 33 k-tiles, runs of unequal length
]


@pytest.mark.parametrize("M,N,K,variant", [p[:4] for p in PRODUCTS])
def test_wide_tiles_same_bits_as_register_staged_and_fp64(M, N, K, variant):
    g = torch.Generator().manual_seed(M + N + K + variant)
    A = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    W = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16).cuda()
    outs = []
    for no_direct in (0, 8):
        out = torch.full((M, N), 0.5, dtype=torch.bfloat16 if variant == 3 else torch.float32, device="cuda")
        tsd.bench_gemm(A, W, out=out, variant=variant + no_direct)
        torch.cuda.synchronize()
        outs.append(out.cpu())
    assert torch.equal(outs[0], outs[1]), f"{(outs[0].float() - outs[1].float()).abs().max():.3e}"
    rows = torch.cat([torch.arange(0, 300), torch.arange(M - 300, M)])
    a, w = A.cpu().double()[rows], W.cpu().double()
    ref = a @ w.T
    if variant in (1, 3):
        ref = ref * torch.rsqrt((a * a).mean(-1, keepdim=True) + 1e-6)
    if variant == 3:
        ref = torch.nn.functional.gelu(ref, approximate="tanh")
    if variant == 2:
        ref = ref + 0.5
    err = (outs[0][rows].double() - ref).abs().max() / ref.abs().max()
    # fp32 accumulation: sqrt(K) roundings of 2^-24 with a factor for the growing partial sums; a bf16 result adds 2^-9
    assert err < (6e-3 if variant == 3 else 2e-6 * K ** 0.5), f"{err:.3e}"


@pytest.mark.parametrize("D,heads,B,N,tile", [
    (512, 8, 128, 72, 2257), (512, 8, 155, 72, 2129), (512, 8, 75, 72, 2128), (512, 8, 40, 40, 2127),   # head_dim 64, every shape
    (512, 16, 128, 72, 2128), (256, 8, 70, 72, 2127), (256, 16, 128, 72, 2128), (256, 16, 65, 72, 2127),  # head_dim 32 and 16
])
def test_rotary_epilogue_same_bits_as_register_staged(D, heads, B, N, tile):
    """The QKV product of a context pass writes queries and the paged cache; what the next round reads of them must not depend on the tile."""
    P, T, K = 16, 3, 2
    m = ModelCfg(1, D, heads, 2 * D)
    g = torch.Generator().manual_seed(D + heads + B)
    n = P * D + (2 * D + 4 * D * D + 4 * D * D) + D + D * P
    w = (torch.randn(n, generator=g) * 0.05).bfloat16().float()
    series = torch.randn(B, N * P, generator=g)
    res, used = [], []
    for flags in (0, tsd.TSD_FLAG_NO_WIDE_GEMM):
        sess = tsd.Session(tsd.make_config(m, m, P, K, B, N + T + K, "bf16", 1.0, seed=3, flags=flags | tsd.TSD_FLAG_SCRAMBLE_PAGES))
        for which in (tsd.TSD_TARGET, tsd.TSD_DRAFT):
            sess.load_weights(which, w.cuda())
        sess.profile_begin(QKV)
        sess.prefill(series.cuda(), N, T * P)
        sess.profile_end()
        used.append({r["tile"] for r in sess.profile_launches()})
        sess.round()
        io = sess.get_round_io()
        res.append({k: io[k].cpu() for k in ("X", "mu_p")})
        sess.close()
    assert tile in used[0] and not any(t > 2000 for t in used[1]), used
    for k in res[0]:
        assert torch.isfinite(res[0][k]).all() and torch.equal(res[0][k], res[1][k]), k


@pytest.mark.parametrize("D,F,E,k,B", [(256, 1024, 8, 2, 640), (512, 1024, 3, 1, 690)])
def test_grouped_products_on_256_row_maps_same_bits_as_register_staged(D, F, E, k, B):
    """A context pass of 12800 / 13800 rows: both products of the experts on maps of 256 rows, last tiles of any length."""
    P, N, T, K = 16, 21, 2, 2
    target, draft = ModelCfg(1, D, D // 64, F, E, k), ModelCfg(1, 64, 1, 256)
    g = torch.Generator().manual_seed(D + E)
    n = lambda m: P * m.d_model + 2 * m.d_model + 4 * m.d_model ** 2 + m.d_model + m.d_model * P + (
        m.d_model * m.n_experts + m.n_experts * 2 * m.d_model * m.d_ff if m.n_experts else 2 * m.d_model * m.d_ff)
    w = [(torch.randn(n(m), generator=g) * 0.05).bfloat16().float() for m in (target, draft)]
    series = torch.randn(B, N * P, generator=g)
    res, used = [], []
    for flags in (0, tsd.TSD_FLAG_NO_WIDE_GEMM):
        sess = tsd.Session(tsd.make_config(target, draft, P, K, B, N + T + K, "bf16", 1.0, seed=3, flags=flags))
        sess.load_weights(tsd.TSD_TARGET, w[0].cuda())
        sess.load_weights(tsd.TSD_DRAFT, w[1].cuda())
        sess.profile_begin(9)  # TSD_K_COUNT
        sess.prefill(series.cuda(), N, T * P)
        sess.profile_end()
        # the experts' products: their rows are the assignments
        used.append({(r["kernel_class"], r["tile"]) for r in sess.profile_launches() if r["model"] == tsd.TSD_TARGET
                     and r["M"] == B * (N - 1) * k and (r["kernel_class"] == GELU or r["K"] == F)})
        sess.round()
        io = sess.get_round_io()
        res.append({x: io[x].cpu() for x in ("X", "mu_p")})
        sess.close()
    assert used[0] == {(GELU, 2257), (RESID, 2256)} and len(used[1]) == 2 and not any(t > 2000 for _, t in used[1]), used
    for x in res[0]:
        assert torch.isfinite(res[0][x]).all() and torch.equal(res[0][x], res[1][x]), x
