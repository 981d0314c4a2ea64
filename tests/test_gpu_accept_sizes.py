"""The acceptance kernel at the edges of its split (four wavefronts over positions, 64 lanes over a patch): statistics against
float64, decisions, committed rows, and what lies behind them, untouched or zeroed; and what the Python call returns."""
import io

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


@pytest.mark.parametrize("B,K,P", [(1, 1, 8), (37, 1, 24), (5, 16, 16), (1023, 6, 96)])
@pytest.mark.parametrize("taps", [True, False])
def test_returned_tensors(B, K, P, taps):
    """What the call returns is what the C entry writes into buffers of one's own; the counts and the patches have memory of
    their own, and all of it can be saved and loaded."""
    g = torch.Generator(device="cuda").manual_seed(B + K)
    mu_q = torch.randn(B, K, P, generator=g, device="cuda")
    X, mu_p = mu_q + 0.2 * torch.randn(B, K, P, generator=g, device="cuda"), torch.randn(B, K + 1, P, generator=g, device="cuda")
    mu_p[:, :K] = mu_q + 0.5 * mu_p[:, :K]
    rounds = torch.arange(B, dtype=torch.int32, device="cuda")
    want = dict(n_acc=torch.full((B,), -7, dtype=torch.int32, device="cuda"), commit=torch.full((B, K + 1, P), 5.0, device="cuda"),
                ell=torch.full((B, K), 5.0, device="cuda"), logu=torch.full((B, K), 5.0, device="cuda"))
    rc = tsd.lib().tsd_accept_commit_static(X.data_ptr(), mu_q.data_ptr(), mu_p.data_ptr(), rounds.data_ptr(), B, K, P, 0.9, 0.7, 0.0, 3,
                                            tsd.binding.TSD_FLAG_CLEAR_REST, *(t.data_ptr() for t in want.values()), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    got = tsd.accept_commit_static(X, mu_q, mu_p, 0.9, 0.7, rounds=rounds, seed=3, want_taps=taps)
    if not taps:
        want["ell"] = want["logu"] = None
    buf = io.BytesIO()
    torch.save(got, buf)
    buf.seek(0)
    loaded = torch.load(buf, weights_only=True)
    assert list(got) == list(loaded) == list(want)
    for name, w in want.items():
        if w is None:
            assert got[name] is None and loaded[name] is None
            continue
        assert got[name].dtype == w.dtype and got[name].is_contiguous() and got[name].device == X.device
        np.testing.assert_array_equal(got[name].cpu().numpy(), w.cpu().numpy())
        np.testing.assert_array_equal(loaded[name].cpu().numpy(), w.cpu().numpy())
    for name in ("n_acc", "commit"):
        assert got[name].untyped_storage().nbytes() == got[name].numel() * 4


def test_no_memory_for_the_outputs():
    """What torch raises where it has no memory (16 TB here), from before any launch."""
    X = torch.zeros(1, 1, 1, device="cuda").expand(1 << 22, 16, 1 << 16)
    with pytest.raises(torch.OutOfMemoryError):
        tsd.accept_commit_static(X, X, X, 1.0)
