"""The acceptance kernel at the edges of its split (four wavefronts over positions, 64 lanes over a patch): statistics against
float64, decisions, committed rows, and what lies behind them, untouched or zeroed."""
import numpy as np
import pytest
import torch

import paper_2511_18191_amd as tsd
from oracle import tsd_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,P", [(1, 8), (3, 64), (4, 72), (5, 96), (8, 136), (9, 16), (16, 256), (13, 1024)])
@pytest.mark.parametrize("clear", [False, True])
def test_static_acceptance(K, P, clear):
    B, sp, sq, seed, r = 37, 0.9, 0.7, 11, 3
    rng = np.random.default_rng(K * 1000 + P)
    mu_p = rng.standard_normal((B, K + 1, P)).astype(np.float32)
    mu_q = (mu_p[:, :K] + 0.5 * rng.standard_normal((B, K, P))).astype(np.float32)
    X = (mu_q + 0.2 * rng.standard_normal((B, K, P))).astype(np.float32)
    dX, dq, dp = (torch.from_numpy(a).cuda() for a in (X, mu_q, mu_p))
    rounds = torch.full((B,), r, dtype=torch.int32, device="cuda")
    n_acc = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    commit = torch.full((B, K + 1, P), 5.0, device="cuda")
    ell, logu = torch.zeros(2, B, K, device="cuda").unbind(0)
    flags = tsd.binding.TSD_FLAG_CLEAR_REST if clear else 0
    rc = tsd.lib().tsd_accept_commit_static(dX.data_ptr(), dq.data_ptr(), dp.data_ptr(), rounds.data_ptr(), B, K, P, sp, sq, 0.0, seed, flags,
                                            n_acc.data_ptr(), commit.data_ptr(), ell.data_ptr(), logu.data_ptr(),
                                            torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    n_acc, commit, ell, logu = (t.cpu().numpy() for t in (n_acc, commit, ell, logu))
    x64, p64, q64 = X.astype(np.float64), mu_p.astype(np.float64), mu_q.astype(np.float64)
    want = (-((x64 - p64[:, :K]) ** 2).sum(-1) / (2 * sp * sp * P) + ((x64 - q64) ** 2).sum(-1) / (2 * sq * sq * P)
            + 0.5 * np.log(sq * sq / (sp * sp)))
    for b in range(B):
        n = n_acc[b]
        u = np.array([orc.uniform(seed, b, r, i + 1) for i in range(K)])
        ok = np.log(u) <= np.minimum(0.0, want[b])
        near = np.abs(np.log(u) - np.minimum(0.0, want[b])) < 1e-4
        first = int(np.argmin(ok)) if not ok.all() else K
        assert n == first or near[: max(n, first) + 1].any()
        tested = n + (n < K)
        # a sum of P squares in fp32 is within P 2^-24 of exact, relative to the sum of what is added (below 1 per dimension here)
        np.testing.assert_allclose(ell[b, :tested], want[b, :tested], rtol=0, atol=4 * P * 2.0 ** -24)
        assert np.isnan(ell[b, tested:]).all() and np.isnan(logu[b, tested:]).all()
        np.testing.assert_array_equal(commit[b, :n], X[b, :n])
        np.testing.assert_array_equal(commit[b, n], mu_p[b, n])
        np.testing.assert_array_equal(commit[b, n + 1:], 0.0 if clear else 5.0)
