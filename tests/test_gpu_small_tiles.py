"""The 64 x 64 direct-to-LDS tiles (products that leave less than a 128-row tile per compute unit) against the
register-staged tiles, bit for bit, and against float64."""
import ctypes as C

import pytest
import torch

import paper_2511_18191_amd as tsd
from synth import ModelCfg

pytestmark = pytest.mark.gpu


# rows, columns, k, variant of tsd_bench_gemm, the tile they take (tests/test_gemm_tiles.py holds the rule to it)
PRODUCTS = [
    (1, 64, 256, 1, 64), (63, 192, 256, 3, 64), (64, 128, 320, 2, 64), (65, 64, 512, 0, 64),   # shortest contraction (no steady k-tile), ragged rows
    (558, 2304, 768, 1, 64), (65, 2048, 512, 3, 64), (4097, 320, 384, 2, 64),                  # a last tile of one row, columns of no 128-multiple
    (1281, 2048, 512, 3, 127),                                                                 # (one 64 x 64 tile too many: 128 x 64)
    (1025, 1024, 1024, 2, 64), (1030, 1024, 4096, 0, 64), (4160, 448, 1088, 2, 64),            # four runs of k-tiles (one tile more than the split takes)
]


@pytest.mark.parametrize("M,N,K,variant", [p[:4] for p in PRODUCTS])
def test_small_direct_tiles_same_bits_as_register_staged_and_fp64(M, N, K, variant):
    g = torch.Generator().manual_seed(M + N + K + variant)
    A = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    W = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16).cuda()
    outs = []
    for no_wide in (0, 8):
        out = torch.full((M, N), 0.5, dtype=torch.bfloat16 if variant == 3 else torch.float32, device="cuda")
        tsd.bench_gemm(A, W, out=out, variant=variant + no_wide)
        torch.cuda.synchronize()
        outs.append(out.cpu())
    assert torch.equal(outs[0], outs[1]), f"{(outs[0].float() - outs[1].float()).abs().max():.3e}"
    a, w = A.cpu().double(), W.cpu().double()
    ref = a @ w.T
    if variant in (1, 3):
        ref = ref * torch.rsqrt((a * a).mean(-1, keepdim=True) + 1e-6)
    if variant == 3:
        ref = torch.nn.functional.gelu(ref, approximate="tanh")
    if variant == 2:
        ref = ref + 0.5
    err = (outs[0].double() - ref).abs().max() / ref.abs().max()
    # fp32 accumulation: sqrt(K) roundings of 2^-24 with a factor for the growing partial sums; a bf16 result adds 2^-9
    assert err < (6e-3 if variant == 3 else 2e-6 * K ** 0.5), f"{err:.3e}"


@pytest.mark.parametrize("D,F,B", [
    (512, 2048, 33), (512, 2112, 65), (256, 2560, 250), (512, 2048, 896),   # runs of unequal length, a last row tile of one row, most tiles
    (768, 3072, 100), (512, 2048, 897), (512, 2176, 64),                    # ... one tile too many, a last run of 4 k-tiles
    (2048, 256, 97), (2048, 256, 193),                                      # an output projection of K = 2048: two row tiles, too many
])
def test_runs_of_a_contraction_in_workgroups_of_their_own(D, F, B):
    """FFN down of few rows: four workgroups per tile, whichever finishes last adds their sums.  Bit for bit the handle without them, over
    steps launched one by one and replayed (the tiles' counters have to be back at zero every time)."""
    P, N, T, K = 16, 3, 6, 2
    m = ModelCfg(2, D, D // 64, F)
    g = torch.Generator().manual_seed(D + F + B)
    n = P * D + 2 * (2 * D + 4 * D * D + 2 * D * F) + D + D * P
    w = (torch.randn(n, generator=g) * 0.05).bfloat16().float().cuda()
    series = torch.randn(B, N * P, generator=g).cuda()
    res = []
    for flags in (0, tsd.TSD_FLAG_NO_WIDE_GEMM):
        sess = tsd.Session(tsd.make_config(m, ModelCfg(1, 64, 1, 96), P, K, B, N + T + K, "bf16", 1.0, seed=3, flags=flags))
        sess.load_weights(tsd.TSD_TARGET, w)
        sess.load_weights(tsd.TSD_DRAFT, torch.zeros(P * 64 + 2 * 64 + 4 * 64 * 64 + 2 * 64 * 96 + 64 + 64 * P))
        sess.prefill(series, N, T * P)
        sess.profile_begin(3)  # TSD_K_RESID
        sess.target_step()
        sess.profile_end()
        tiles = {r["tile"] for r in sess.profile_launches() if r["K"] == max(D, F)}
        assert tiles == {464 if flags or (B + 63) // 64 * (D // 64) > 112 else 2464}, tiles
        for _ in range(3):
            sess.prefill(series, N, T * P)
            for _ in range(T):
                sess.target_step()
            res.append(sess.get_forecast().cpu())
        sess.close()
    assert torch.isfinite(res[0]).all()
    for other in res[1:]:
        assert torch.equal(res[0], other)


@pytest.mark.parametrize("D,F,B", [(256, 2048, 150), (512, 2048, 90)])
def test_runs_capped_on_the_device_while_series_finish(D, F, B):
    """Rounds without a look at the counts between them: launches sized for the whole batch, rows capped by the count on the device as
    series finish at different times.  Bit for bit the handle that neither compacts nor takes the runs."""
    P, N, T, K = 16, 5, 9, 2
    m = ModelCfg(2, D, D // 64, F)
    g = torch.Generator().manual_seed(D + B)
    w = (torch.randn(P * D + 2 * (2 * D + 4 * D * D + 2 * D * F) + D + D * P, generator=g) * 0.05).bfloat16().float().cuda()
    series = torch.randn(B, N * P, generator=g).cuda()
    res = []
    for flags in (0, tsd.TSD_FLAG_NO_GRAPH, tsd.TSD_FLAG_NO_COMPACT | tsd.TSD_FLAG_NO_WIDE_GEMM):
        sess = tsd.Session(tsd.make_config(m, ModelCfg(1, 64, 1, 96), P, K, B, N + T + K, "bf16", 1.0, seed=3, flags=flags))
        sess.load_weights(tsd.TSD_TARGET, w)
        sess.load_weights(tsd.TSD_DRAFT, torch.zeros(P * 64 + 2 * 64 + 4 * 64 * 64 + 2 * 64 * 96 + 64 + 64 * P))
        sess.set_accept_override(0.5)
        for polled in (True, False):
            sess.prefill(series, N, T * P)
            sess.profile_begin(3)  # TSD_K_RESID
            sess.round()
            sess.profile_end()
            tiles = {r["tile"] for r in sess.profile_launches() if r["K"] == F}
            assert tiles == {464 if flags & tsd.TSD_FLAG_NO_WIDE_GEMM else 2464}, tiles
            left = {sess.num_active()}
            for _ in range(T):
                sess.round()
                if polled:
                    left.add(sess.num_active())
            assert sess.num_active() == 0 and (not polled or len(left) > 3), left
            res.append(sess.get_forecast().cpu())
        sess.close()
    assert torch.isfinite(res[0]).all()
    for other in res[1:]:
        assert torch.equal(res[0], other)


def test_arenas_too_small_for_all_rows_keep_the_runs():
    """The partial sums go after the context's rows: an arena a little short of the full size still takes them, the least one does without."""
    P, N, T, K, B, D, F = 16, 20, 4, 2, 100, 256, 2048
    m, d = ModelCfg(2, D, D // 64, F), ModelCfg(1, 64, 1, 96)
    g = torch.Generator().manual_seed(5)
    w = (torch.randn(P * D + 2 * (2 * D + 4 * D * D + 2 * D * F) + D + D * P, generator=g) * 0.05).bfloat16().float().cuda()
    series = torch.randn(B, N * P, generator=g).cuda()
    sess = tsd.Session(tsd.make_config(m, d, P, K, B, N + T + K, "bf16", 1.0, seed=3))
    full, base = sess.arena_bytes, (sess.arena.data_ptr() + 255) & ~255
    room = 4 * 112 * 64 * 64 * 4 + 512
    rows = (B * (N + T + K) - B * (K + 1)) * (4 * D + 3 * 2 * D + 2 * F + 8)   # what the contexts' rows take beyond a round's
    res = []
    for size, tile in ((full, 2464), (full - 256, 2464), ((full - rows // 2) // 256 * 256, 2464), ((full - rows - room // 2) // 256 * 256, 464)):
        sess.close()
        h = C.c_void_p()
        assert tsd.lib().tsd_create(C.byref(sess.cfg), base, size, C.byref(h)) == 0
        sess.h = h
        sess.load_weights(tsd.TSD_TARGET, w)
        sess.load_weights(tsd.TSD_DRAFT, torch.zeros(P * 64 + 2 * 64 + 4 * 64 * 64 + 2 * 64 * 96 + 64 + 64 * P))
        sess.prefill(series, N, T * P)
        sess.profile_begin(3)  # TSD_K_RESID
        sess.target_step()
        sess.profile_end()
        assert {r["tile"] for r in sess.profile_launches() if r["K"] == F} == {tile}, size
        for _ in range(T - 1):
            sess.target_step()
        res.append(sess.get_forecast().cpu())
    sess.close()
    for other in res:
        assert torch.isfinite(other).all() and torch.equal(res[0], other)
