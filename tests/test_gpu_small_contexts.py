"""Short contexts on small handles (at most 32 decode rows): a series' context has the sums of the skinny products however many others are
prefilled with it, on the skinny kernel itself and on the 64 x 64 tiles that take its place beyond 32 rows."""
import pytest
import torch

import paper_2511_18191_amd as tsd
from synth import ModelCfg

pytestmark = pytest.mark.gpu
FAMILIES = 9  # TSD_K_COUNT


def _models(layers, D, F, g, P):
    m = ModelCfg(layers, D, D // 64, F)
    n = P * D + layers * (2 * D + 4 * D * D + 2 * D * F) + D + D * P
    return m, (torch.randn(n, generator=g) * 0.05).bfloat16().float()


def _session(m, w, P, K, B, tokens, flags=0):
    sess = tsd.Session(tsd.make_config(m, m, P, K, B, tokens, "bf16", 1.0, seed=3, flags=flags))
    for which in (tsd.TSD_TARGET, tsd.TSD_DRAFT):
        sess.load_weights(which, w.cuda())
    return sess


def _first_round(sess, series, N, H):
    sess.profile_begin(FAMILIES)
    sess.prefill(series.cuda(), N, H)
    sess.profile_end()
    tiles = {(r["K"], r["tile"]) for r in sess.profile_launches() if r["kernel_class"] in (1, 3, 4)}  # QKV, residual, GELU
    sess.round()
    io = sess.get_round_io()
    return {k: io[k].cpu() for k in ("X", "mu_p")}, tiles


@pytest.mark.parametrize("B,N,K", [(5, 30, 4), (3, 12, 2), (16, 33, 1)])
def test_context_alone_and_in_company_same_bits(B, N, K):
    P, T = 32, 3
    g = torch.Generator().manual_seed(B + N)
    m, w = _models(2, 512, 2048, g, P)
    series = torch.randn(B, N * P, generator=g)
    sess = _session(m, w, P, K, B, N + T + K)
    together, _ = _first_round(sess, series, N, T * P)
    for b in {0, 1, B - 1}:
        alone, _ = _first_round(sess, series[b:b + 1], N, T * P)
        for k in alone:
            assert torch.isfinite(alone[k][0]).all() and torch.equal(alone[k][0], together[k][b]), (b, k)
    sess.close()


@pytest.mark.parametrize("B,N,K,D,F,down", [
    (3, 12, 2, 512, 2048, 16),      # 33 rows, 16 shares of one step; the down product stays with the skinny kernel
    (2, 33, 2, 256, 1088, 2016),    # 64 rows, four shares; 34 steps in shares of three, the last one short, some empty
    (5, 14, 2, 768, 3072, 2016),    # 65 rows, shares of two steps and of six
    (16, 33, 1, 512, 2048, 2016),   # 512 rows, shares of four
    (7, 20, 3, 320, 1024, 2016),    # 133 rows, widths of an odd number of tiles, ten steps in four shares
])
def test_tiles_with_the_skinny_products_sums(B, N, K, D, F, down):
    P, T = 32, 3
    g = torch.Generator().manual_seed(B + N + D + F)
    m, w = _models(2, D, F, g, P)
    series = torch.randn(B, N * P, generator=g)
    res, used = [], []
    for flags in (0, tsd.TSD_FLAG_NO_WIDE_GEMM):
        sess = _session(m, w, P, K, B, N + T + K, flags=flags | tsd.TSD_FLAG_SCRAMBLE_PAGES)
        io, tiles = _first_round(sess, series, N, T * P)
        res.append(io)
        used.append(tiles)
        sess.close()
    assert used == [{(D, 2016), (F, down)}, {(D, 16), (F, 16)}], used
    for k in res[0]:
        assert torch.isfinite(res[0][k]).all() and torch.equal(res[0][k], res[1][k]), k
