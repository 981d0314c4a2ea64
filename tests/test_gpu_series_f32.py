"""Small fp32 models run a series per workgroup (series_f32.hip): bit for bit the kernels it replaces, which the same handle takes under a
measurement, over the sizes where its indexing changes: 1 to 17 rows per pass, every width and head size, patches that leave blocks
and k-runs partly filled, pages of one token, more series than fit the grid's first turn, contexts of one and several blocks of 32 and
of 16 rows; values that are none, a caller's capture, two handles at once."""
import threading

import numpy as np
import pytest
import torch

import paper_2511_18191_amd as tsd
from harness import TOL, Case, lockstep
from synth import ModelCfg

pytestmark = pytest.mark.gpu

T64, D32 = ModelCfg(2, 64, 4, 256), ModelCfg(1, 32, 2, 128)


def forecasts(case, sess, kernel_by_kernel, steps):
    c = case.cfg
    if kernel_by_kernel:
        sess.profile_begin(3)  # TSD_K_RESID
    sess.prefill(case.context, c.n_ctx, c.horizon)
    sess.run_rounds()
    out = [sess.get_forecast().cpu().numpy(), sess.get_series_stats().cpu().numpy()]
    sess.reset_decode()
    for _ in range(steps):
        sess.target_step()
    out.append(sess.get_forecast().cpu().numpy())
    if kernel_by_kernel:
        sess.profile_end()
    return out


def m(L, D, H):
    return ModelCfg(L, D, H, 4 * D)


@pytest.mark.parametrize("B,K,target,draft,P,N,T", [
    (8, 4, T64, D32, 16, 32, 6), (1, 1, T64, D32, 16, 4, 3), (3, 15, T64, D32, 8, 17, 18), (2, 16, m(1, 64, 2), m(2, 32, 1), 24, 18, 19),  # 2, 16, 17 rows
    (5, 3, m(3, 128, 2), m(1, 64, 2), 32, 40, 5), (4, 2, m(1, 128, 4), m(2, 64, 1), 40, 34, 5),    # 24 blocks, a patch of two and a half k-runs
    (2, 2, m(1, 128, 8), m(1, 128, 2), 200, 50, 4), (2, 16, m(2, 64, 2), m(1, 64, 4), 16, 125, 18), (3, 6, m(2, 128, 2), D32, 16, 50, 12),  # twelve and a half; 124 tokens
    (40, 2, T64, D32, 16, 12, 7), (200, 3, m(1, 64, 1), D32, 16, 5, 5), (512, 1, T64, D32, 16, 3, 3),
])
def test_same_bits_as_kernel_by_kernel(B, K, target, draft, P, N, T):
    case = Case("cfg1", B=B, K=K, target=target, draft=draft, patch=P, context=N * P, horizon=T * P - P // 2, random_gains=True)
    sess = case.session()
    got = forecasts(case, sess, False, T)
    ran = sess.resident_passes()
    assert ran >= 2 + T
    ref = forecasts(case, sess, True, T)
    assert sess.resident_passes() == ran
    for g, r in zip(got, ref):
        np.testing.assert_array_equal(g, r)
    again = forecasts(case, sess, False, T)
    for g, r in zip(again, ref):
        np.testing.assert_array_equal(g, r)
    sess.close()


@pytest.mark.parametrize("pages,flags", [(1, 0), (2, tsd.TSD_FLAG_SCRAMBLE_PAGES), (16, tsd.TSD_FLAG_NO_PINNED_COUNTS), (16, tsd.TSD_FLAG_BATCH_SYNC),
                                         (16, tsd.TSD_FLAG_NO_COMPACT), (64, tsd.TSD_FLAG_THRESHOLD_RULE)])
def test_lockstep(pages, flags):
    case = Case("cfg1", B=6, sigma=0.2)
    sess = case.session(page_tokens=pages, flags=flags)
    sync = bool(flags & tsd.TSD_FLAG_BATCH_SYNC)
    rep = lockstep(case, sess, sync=sync, rule="threshold" if flags & tsd.TSD_FLAG_THRESHOLD_RULE else "ratio")
    assert rep["max_rel_X"] <= TOL["fp32"] and rep["max_rel_mu_p"] <= TOL["fp32"], rep
    assert sess.num_active() == 0 and sess.resident_passes() > 0
    got, ref = forecasts(case, sess, False, 2), forecasts(case, sess, True, 2)
    for g, r in zip(got, ref):
        np.testing.assert_array_equal(g, r)
    sess.close()


def test_refill():
    """Slots refilled in the middle of a decode forecast what a batch of their own does."""
    case = Case("cfg1", B=6)
    c = case.cfg
    sess = case.session()
    sess.prefill(case.context, c.n_ctx, c.horizon)
    want = None
    for kernel_by_kernel in (True, False):
        if kernel_by_kernel:
            sess.profile_begin(3)  # TSD_K_RESID
        sess.prefill(case.context, c.n_ctx, c.horizon)
        sess.round()
        sess.refill([4, 1], np.roll(case.context[:2], 7, axis=1))
        sess.run_rounds()
        out = sess.get_forecast().cpu().numpy()
        if kernel_by_kernel:
            sess.profile_end()
            want = out
    np.testing.assert_array_equal(out, want)
    sess.close()


# (the last two: horizons behind which 32 rows at a time do not fit)
@pytest.mark.parametrize("B,target,draft,N,T", [
    (3, T64, D32, 33, 2), (2, T64, D32, 34, 2), (3, m(2, 64, 2), m(1, 64, 1), 65, 2),             # 32, 33 and 64 tokens
    (64, T64, D32, 66, 2), (128, m(1, 64, 2), m(1, 32, 1), 129, 2), (65, m(1, 32, 1), m(1, 32, 2), 97, 1),    # three and four blocks
    (2, m(2, 128, 8), D32, 33, 3), (64, m(1, 128, 2), m(1, 128, 4), 34, 2), (129, m(1, 128, 4), D32, 75, 1),  # one to three of 128
    (600, T64, D32, 10, 2), (512, m(1, 128, 2), m(1, 64, 1), 2, 1),                               # more series than rounds take; one token
    (4, m(1, 128, 2), m(1, 64, 2), 24, 70), (3, T64, m(1, 64, 4), 65, 160),
])
def test_contexts(B, target, draft, N, T):
    """Contexts this kernel takes, on a new handle and on freed slots: one launch each, then forecasts with the same bits."""
    case = Case("cfg1", B=B, K=2, target=target, draft=draft, patch=16, context=N * 16, horizon=T * 16, random_gains=True)
    c, P = case.cfg, 16
    sess = case.session()
    newcomers = list(range(B - 1, -1, -1)) if (N - 1 > 64 or target.d_model == 128) else [B - 1]   # (as many as the rule asks for)
    other = np.roll(case.context, 5, axis=1)[:len(newcomers)]
    out = []
    for kernel_by_kernel in (False, True):
        passes = [sess.resident_passes()]
        if kernel_by_kernel:
            sess.profile_begin(3)  # TSD_K_RESID
        sess.prefill(case.context, N, c.horizon)
        passes.append(sess.resident_passes())
        sess.run_rounds(2)
        out.append(sess.get_forecast().cpu().numpy())
        passes.append(sess.resident_passes())
        sess.refill(newcomers, other)
        passes.append(sess.resident_passes())
        sess.round()
        out.append(sess.get_round_io())
        out.append(sess.get_forecast().cpu().numpy())
        if kernel_by_kernel:
            sess.profile_end()
        grown = np.diff(passes).tolist()
        if kernel_by_kernel:
            assert grown == [0, 0, 0]
        else:
            assert grown[0] == 1 and grown[2] == 1 and (grown[1] > 0) == (B <= 512)
    for g, r in zip(out[:3], out[3:]):
        if isinstance(g, dict):
            for name in g:
                np.testing.assert_array_equal(g[name].cpu().numpy(), r[name].cpu().numpy(), err_msg=name)
        else:
            assert np.isfinite(g).any()
            np.testing.assert_array_equal(g, r)
    sess.close()


@pytest.mark.parametrize("B", [257, 512, 1500])
def test_list_of_active_series(B):
    """Several trips of the compaction, inside a round and as a kernel of its own: whoever still decodes is on the list once, so that
    every decode ends where one without a list does."""
    case = Case("cfg1", B=B, K=2, target=m(1, 32, 1), draft=m(1, 32, 2), patch=16, context=6 * 16, horizon=7 * 16, sigma=0.15)
    c = case.cfg
    sess, ref = case.session(), case.session(flags=tsd.TSD_FLAG_NO_COMPACT)
    for s in (sess, ref):
        s.prefill(case.context, c.n_ctx, c.horizon)
    counts = []
    while not counts or counts[-1]:
        for s in (sess, ref):
            s.round()
        counts.append(sess.num_active())
        committed = sess.get_state()["committed"]
        np.testing.assert_array_equal(committed.cpu().numpy(), ref.get_state()["committed"].cpu().numpy())
        assert counts[-1] == int((committed < c.T).sum())
    assert any(0 < n < B for n in counts)
    np.testing.assert_array_equal(sess.get_forecast().cpu().numpy(), ref.get_forecast().cpu().numpy())
    for s in (sess, ref):
        s.close()


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("K,target", [(9, T64), (16, T64), (16, m(1, 32, 1)), (12, m(2, 128, 2))])
def test_values_that_are_none(bad, K, target):
    """A proposal that is not finite spoils what sees it and nothing else: the verification of more than eight tokens goes through the
    matrix cores, whose products of weight 0 must not reach the tokens before it (nor change their bits)."""
    B, at = 5, 4
    case = Case("cfg1", B=B, K=K, target=target, draft=D32, patch=16, context=20 * 16, horizon=24 * 16)
    c = case.cfg
    sess = case.session()
    sess.prefill(case.context, c.n_ctx, c.horizon)
    sess.draft_propose()
    sess.sync()
    io = sess.get_round_io()
    X = io["X"].clone()
    X[1, at] = bad
    X[3, at, 7] = bad
    got = []
    for proposals in (io["X"], X, io["X"]):
        ran = sess.resident_passes()
        sess.set_round_io(proposals, io["mu_q"], io["mu_p"])
        sess.target_verify()
        got.append(sess.get_round_io()["mu_p"].cpu().numpy())
        assert sess.resident_passes() - ran == 1
    assert np.isfinite(got[0]).all()
    np.testing.assert_array_equal(got[0], got[2])
    for b in range(B):
        spoilt = at + 1 if b in (1, 3) else K + 1   # (row 0 is the pending token's)
        np.testing.assert_array_equal(got[1][b, :spoilt], got[0][b, :spoilt])
        assert not np.isfinite(got[1][b, spoilt:]).any()
    sess.close()


def test_a_caller_captures_a_forecast():
    """Context, rounds and forecast in a graph of the caller's, replayed over other series, with eager work in between."""
    case = Case("cfg1", B=6)
    c = case.cfg
    sess, fresh = case.session(), case.session()
    series = torch.from_numpy(case.context).cuda()
    out = torch.empty(6, c.horizon, device="cuda")
    L, h, raw = tsd.lib(), sess.h, sess.stream.cuda_stream
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=sess.stream, capture_error_mode="thread_local"):
        rc = [L.tsd_prefill(h, series.data_ptr(), 6, c.n_ctx, c.horizon, raw)]
        rc += [L.tsd_round(h, raw) for _ in range(c.T)]      # (a round commits at least one patch)
        rc.append(L.tsd_get_forecast(h, out.data_ptr(), raw))
    assert not any(rc) and sess.resident_passes() == 1 + c.T
    for i in range(4):
        ctx = np.roll(case.context, 3 * i, axis=1)
        series.copy_(torch.from_numpy(ctx))
        torch.cuda.synchronize()
        with torch.cuda.stream(sess.stream):
            graph.replay()
        fresh.prefill(ctx, c.n_ctx, c.horizon)
        fresh.run_rounds()
        want = fresh.get_forecast().cpu().numpy()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), want)
    sess.close()
    fresh.close()


def test_two_handles_at_once():
    """On two streams from one thread, launch after launch, and in two threads: the results of a handle alone."""
    cases = [Case("cfg1", B=40), Case("cfg1", B=300, target=m(1, 128, 4), draft=m(1, 64, 2))]
    sess, want, errors = [k.session() for k in cases], [], []
    assert sess[0].stream != sess[1].stream

    def start(k, s):
        s.prefill(k.context, k.cfg.n_ctx, k.cfg.horizon)

    for k, s in zip(cases, sess):
        start(k, s)
        s.run_rounds()
        want.append(s.get_forecast().cpu().numpy())

    def work(k, s, w):
        try:
            for _ in range(5):
                start(k, s)
                s.run_rounds()
                np.testing.assert_array_equal(s.get_forecast().cpu().numpy(), w)
        except Exception as e:
            errors.append(e)

    for k, s in zip(cases, sess):
        start(k, s)
    for _ in range(max(k.cfg.T for k in cases)):
        for s in sess:
            s.round()
    for s, w in zip(sess, want):
        np.testing.assert_array_equal(s.get_forecast().cpu().numpy(), w)
    threads = [threading.Thread(target=work, args=a) for a in zip(cases, sess, want)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for s in sess:
        s.close()
