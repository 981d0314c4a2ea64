"""bf16 attention off the matrix cores (head_dim 16 and 32, pages of fewer than 8 tokens): a wavefront per query, which few series take, against
a wavefront per (series, head), which the same series take among many, to the bit."""
import pytest
import torch

import paper_2511_18191_amd as tsd
from synth import ModelCfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,heads,N,K,page", [
    (64, 4, 20, 4, 16), (64, 2, 10, 1, 16),    # head_dim 16 and 32; contexts of 19 queries, chunks of 8, 8 and 3, and of 9
    (128, 2, 9, 7, 4), (128, 4, 34, 8, 2),     # head_dim 64 on small pages, a whole chunk; 32: more queries than a chunk in the decode too
])
def test_bf16_series_alone_and_among_many_same_bits(D, heads, N, K, page):
    P, T = 16, 5
    many = 2100 // heads                       # 2048 (series, heads) are the most that take a wavefront per query
    m = ModelCfg(2, D, heads, 4 * D)
    g = torch.Generator().manual_seed(D + heads + N)
    n = P * D + 2 * (2 * D + 4 * D * D + 8 * D * D) + D + D * P
    w = (torch.randn(n, generator=g) * 0.05).bfloat16().float()
    series = torch.randn(many, N * P, generator=g)
    res = []
    for B in (3, many):
        # (the skinny products of small handles sum k in another order, the one-launch draft has its own attention)
        sess = tsd.Session(tsd.make_config(m, m, P, K, B, N + T + K, "bf16", 1.0, seed=3, page_tokens=page,
                                           flags=tsd.TSD_FLAG_NO_SKINNY | tsd.TSD_FLAG_NO_FUSED_DRAFT))
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
