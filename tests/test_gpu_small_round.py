"""Decode passes of at most 32 rows run as one resident kernel: lock-step with the oracle, and bit for bit the kernels it
replaces, over the sizes where its indexing changes (row tiles of 4, 8, 16 and 2 x 16, 4, 8 and 16 columns per workgroup, workers
with fewer than four slabs, patches that are no whole k-step, more cached keys than are fetched together), and two handles at a
time.  Every case asserts that the one side ran on that kernel and the other did not."""
import threading

import numpy as np
import pytest
import torch

import paper_2511_18191_amd as tsd
from harness import TOL, Case, lockstep
from synth import ModelCfg

pytestmark = pytest.mark.gpu

D1 = ModelCfg(1, 64, 1, 96)


@pytest.mark.parametrize("B,K,target,draft,P,N,T", [
    (1, 1, None, None, 96, 6, 3), (2, 1, None, None, 96, 6, 3), (1, 4, None, None, 96, 6, 6), (1, 15, None, None, 96, 6, 20),
    (2, 15, None, None, 96, 6, 18), (16, 1, None, None, 96, 6, 3), (8, 3, None, None, 96, 6, 5),   # 2 .. 32 rows
    (3, 4, ModelCfg(2, 192, 3, 288), D1, 48, 5, 6),                # 6 and 9 k-steps (three slabs), a patch of one and a half
    (5, 2, ModelCfg(1, 384, 6, 1536), ModelCfg(2, 128, 2, 192), 16, 4, 5),      # 8 columns, 15 rows
    (2, 4, ModelCfg(1, 1024, 16, 4096), ModelCfg(1, 384, 6, 1536), 96, 4, 6),   # the widest products it takes, 10 rows
    # 8 and 16 columns at 2, 6, 15 and 30 rows, two layers of both models
    (1, 1, ModelCfg(2, 384, 6, 1536), ModelCfg(2, 384, 6, 768), 32, 4, 4), (1, 1, ModelCfg(2, 768, 12, 3072), D1, 96, 4, 3),
    (2, 2, ModelCfg(2, 384, 6, 1536), ModelCfg(2, 512, 8, 1024), 96, 4, 5), (2, 2, ModelCfg(2, 768, 12, 3072), D1, 112, 4, 5),
    (3, 4, ModelCfg(2, 512, 8, 2048), ModelCfg(2, 384, 6, 1536), 96, 4, 6), (3, 4, ModelCfg(2, 896, 14, 3584), D1, 96, 4, 6),
    (5, 5, ModelCfg(2, 512, 8, 2048), ModelCfg(2, 256, 4, 1024), 96, 4, 7), (5, 5, ModelCfg(2, 1024, 16, 4096), ModelCfg(2, 384, 6, 1536), 96, 4, 7),
    (2, 3, ModelCfg(2, 256, 4, 512), D1, 560, 4, 5),               # an embedding of 17 and a half k-steps, two per slab
    (2, 3, ModelCfg(1, 128, 2, 256), D1, 16, 300, 5),              # ten 32-key steps, four at a time
])
def test_lockstep(B, K, target, draft, P, N, T):
    over = dict(patch=P, context=N * P)
    if target:
        over.update(target=target, draft=draft)
    case = Case("mini2", B=B, K=K, horizon=T * P, random_gains=True, **over)
    sess = case.session()
    # (proposal 15 is the end of a chain of 15 bf16 passes, each within PASS_TOL = 8e-3 of exact on its own inputs, which lockstep
    #  asserts for every one of them; independent roundings add up to 8e-3 sqrt(15) = 3.1e-2, twice that is allowed)
    tol = TOL["bf16"] if K < 15 else 6e-2
    # (PASS_TOL is a bound on whole patches; the largest relative error over patches of 16 values spreads further: 8.42e-3 here and
    #  8.42e-3 kernel by kernel)
    rep = lockstep(case, sess, tol=tol, per_pass=P > 16)
    assert rep["max_rel_X"] <= tol and rep["max_rel_mu_p"] <= tol, rep
    # a whole forecast and the target-only steps: the same bits as kernel by kernel (a handle without pinned host words)
    ref = case.session(flags=tsd.TSD_FLAG_NO_PINNED_COUNTS)
    for s in (sess, ref):
        s.prefill(case.context, case.cfg.n_ctx, case.cfg.horizon)
        s.run_rounds()
    np.testing.assert_array_equal(sess.get_forecast().cpu().numpy(), ref.get_forecast().cpu().numpy())
    for s in (sess, ref):
        s.reset_decode()
        for _ in range(T):
            s.target_step()
    np.testing.assert_array_equal(sess.get_forecast().cpu().numpy(), ref.get_forecast().cpu().numpy())
    # two launches per lock-step round, one per round, one per target step
    assert sess.resident_passes() >= 2 * rep["rounds"] + (T + K) // (K + 1) + T and ref.resident_passes() == 0
    sess.close()
    ref.close()


W192, W640, W960 = ModelCfg(2, 192, 3, 384), ModelCfg(2, 640, 10, 2560), ModelCfg(2, 960, 15, 3840)


@pytest.mark.parametrize("B,K,target,draft", [
    (8, 3, W192, W192), (8, 3, W640, W192), (4, 7, W960, W640), (2, 15, W640, W192), (16, 1, W192, W640), (2, 15, W960, W960)])
def test_32_rows_with_partly_used_workers(B, K, target, draft):
    """Passes of exactly 32 rows through products whose last worker has fewer than four slabs (6, 20 and 30 k-steps; 4, 8 and 16
    columns per workgroup): a read past the end of row 31 would fetch lines that the same stage publishes."""
    P, N, T = 96, 5, 2 * K + 3
    case = Case("mini2", B=B, K=K, patch=P, context=N * P, horizon=T * P, random_gains=True, target=target, draft=draft)
    out = []
    for s in (case.session(), case.session(flags=tsd.TSD_FLAG_NO_PINNED_COUNTS)):
        for _ in range(2):      # the second forecast finds the first one's exchange buffer
            s.prefill(case.context, case.cfg.n_ctx, case.cfg.horizon)
            s.run_rounds()
        out.append(s.get_forecast().cpu().numpy())
        assert (s.resident_passes() > 0) == (len(out) == 1)
        s.close()
    np.testing.assert_array_equal(*out)


def test_two_handles_on_two_streams():
    """Rounds of two handles enqueued alternately without waiting give what each gives alone, and only the one that is alone
    on the GPU takes the resident kernel."""
    cases = [Case("mini2", B=2), Case("mini3", B=3)]
    alone = []
    for c in cases:
        s = c.session()
        s.prefill(c.context, c.cfg.n_ctx, c.cfg.horizon)
        s.run_rounds()
        alone.append(s.get_forecast().cpu().numpy())
        s.close()
    sess = [c.session() for c in cases]
    for c, s in zip(cases, sess):
        s.prefill(c.context, c.cfg.n_ctx, c.cfg.horizon)
    torch.cuda.synchronize()
    for _ in range(20):            # (a few milliseconds of work; the next call comes a fraction of one later)
        sess[0].reset_decode()
        sess[0].round()
    assert sess[0].resident_passes() == 20
    sess[1].round()
    assert sess[1].resident_passes() == 0      # the other stream's passes are in flight: kernel by kernel, the GPU shared
    torch.cuda.synchronize()
    sess[1].round()
    assert sess[1].resident_passes() == 1
    for s in sess:
        s.reset_decode()
    for _ in range(max(c.cfg.T for c in cases)):      # a round commits at least one patch
        for s in sess:
            s.round()
    for s, ref in zip(sess, alone):
        assert s.num_active() == 0
        np.testing.assert_array_equal(s.get_forecast().cpu().numpy(), ref)
        s.close()


def test_two_handles_in_two_threads():
    """Two programs' worth of forecasts at once, on fresh handles each time so that either thread captures its launches while the other
    looks whether it may take the resident kernel: no error, and the results of a handle alone."""
    case = Case("mini2", B=2)
    c = case.cfg
    ref = case.session()
    want = []
    for target_only in (False, True):
        ref.prefill(case.context, c.n_ctx, c.horizon)
        for _ in range(c.T):
            ref.target_step() if target_only else ref.round()
        want.append(ref.get_forecast().cpu().numpy())
    ref.close()
    errors = []

    def work(s):
        try:
            for i in range(6):
                s.prefill(case.context, c.n_ctx, c.horizon)
                for _ in range(c.T):
                    s.target_step() if i % 2 else s.round()
                np.testing.assert_array_equal(s.get_forecast().cpu().numpy(), want[i % 2])
        except Exception as e:
            errors.append(e)

    for _ in range(4):
        sess = [case.session() for _ in range(2)]
        threads = [threading.Thread(target=work, args=(s,)) for s in sess]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for s in sess:
            s.close()
    assert not errors, errors


def test_beside_a_large_batch():
    """A handle of any kind that is busy on another stream keeps a small one off the resident kernel; on the same stream, which
    orders the two, it does not."""
    big, small = Case("mini2", B=64), Case("mini2", B=2)
    sb, ss = big.session(), small.session()
    for c, s in ((big, sb), (small, ss)):
        s.prefill(c.context, c.cfg.n_ctx, c.cfg.horizon)
    torch.cuda.synchronize()
    ss.round()                     # (others' passes are watched while somebody asks, i.e. has asked in the last 100 ms)
    assert ss.resident_passes() == 1
    for _ in range(20):
        sb.reset_decode()
        sb.round()
    assert sb.resident_passes() == 0
    ss.round()
    assert ss.resident_passes() == 1
    torch.cuda.synchronize()
    ss.reset_decode()
    ss.stream = sb.stream
    torch.cuda.synchronize()
    for _ in range(20):
        sb.reset_decode()
        sb.round()
    ss.run_rounds()
    assert ss.resident_passes() > 1
    got = ss.get_forecast().cpu().numpy()
    ref = small.session(flags=tsd.TSD_FLAG_NO_PINNED_COUNTS)
    ref.prefill(small.context, small.cfg.n_ctx, small.cfg.horizon)
    ref.run_rounds()
    np.testing.assert_array_equal(got, ref.get_forecast().cpu().numpy())
    for s in (sb, ss, ref):
        s.close()


def test_a_capture_of_the_callers_goes_on():
    """Rounds of two handles while the caller captures a stream of its own, in the mode that refuses most: the look at the other
    handle's passes must not end the capture."""
    case = Case("mini2", B=2)
    c = case.cfg
    sess = [case.session() for _ in range(2)]
    want = []
    for s in sess:
        s.prefill(case.context, c.n_ctx, c.horizon)
        s.run_rounds()
        want.append(s.get_forecast().cpu().numpy())
        s.reset_decode()
    torch.cuda.synchronize()
    x = torch.zeros(8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    # (torch deals its streams out of a ring of 32: the one it captures on by default may be a session's)
    own = torch.cuda.Stream()
    while own.cuda_stream in [s.stream.cuda_stream for s in sess]:
        own = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=own, capture_error_mode="global"):
        x += 1
        for _ in range(c.T):
            for s in sess:
                assert tsd.lib().tsd_round(s.h, s.stream.cuda_stream) == 0
        x += 1
    torch.cuda.synchronize()
    for s, w in zip(sess, want):
        assert s.num_active() == 0
        np.testing.assert_array_equal(s.get_forecast().cpu().numpy(), w)
        s.close()
    for n in (1, 2, 3):
        graph.replay()
        assert x.cpu().tolist() == [2.0 * n] * 8


@pytest.mark.parametrize("B,K,target,draft,P,N", [
    (1, 4, None, None, 96, 6), (16, 1, W192, W640, 96, 5), (2, 15, W640, W192, 96, 5),
    (3, 4, ModelCfg(2, 192, 3, 288), D1, 48, 5), (2, 3, ModelCfg(2, 768, 12, 3072), ModelCfg(2, 384, 6, 1536), 560, 4),
    (2, 3, ModelCfg(1, 128, 2, 256), D1, 16, 300)])
def test_a_launch_that_gives_up_is_finished_alone(B, K, target, draft, P, N):
    """A launch whose workgroups do not wait for one another is finished by one workgroup: the same bits, no error to miss, and the
    handle runs kernel by kernel afterwards."""
    over = dict(patch=P, context=N * P, horizon=(2 * K + 3) * P)
    if target:
        over.update(target=target, draft=draft)
    case = Case("mini2", B=B, K=K, random_gains=True, **over)
    c = case.cfg
    T = 2 * K + 3

    def decode(s, give_up_at):
        """A forecast call by call; from call `give_up_at` on the launches do not wait."""
        out, calls = [], [s.draft_propose, s.target_verify, s.accept_commit, s.round, s.round]
        s.prefill(case.context, c.n_ctx, c.horizon)
        for i, call in enumerate(calls):
            if i == give_up_at:
                s.set_resident_wait(0)
            before = s.resident_passes()
            call()
            if i == give_up_at:
                assert s.resident_passes() == before + 1
            s.sync()
            io = s.get_round_io()
            out += [io[k].cpu().numpy() for k in (("X",), ("X", "mu_p"), io, io, ())[i]]      # (what this call is sure to have written)
        n = s.resident_passes()
        for _ in range(3):                   # rounds enqueued without looking, then the rest
            s.round()
        s.run_rounds()
        assert give_up_at is None or s.resident_passes() == n
        return out + [s.get_forecast().cpu().numpy()]

    ref = case.session(flags=tsd.TSD_FLAG_NO_PINNED_COUNTS)
    want = decode(ref, None)
    ref.close()
    for give_up_at in (0, 1, 3, 4):          # draft steps, verification, a round, a round that follows the device's counts
        s = case.session()
        for a, b in zip(decode(s, give_up_at), want):
            np.testing.assert_array_equal(a, b)
        s.close()
    # a whole forecast enqueued before anybody looks
    for s in (case.session(), case.session(flags=tsd.TSD_FLAG_NO_PINNED_COUNTS)):
        s.set_resident_wait(0)
        s.prefill(case.context, c.n_ctx, c.horizon)
        for _ in range(T):
            s.target_step()
        want.append(s.get_forecast().cpu().numpy())
        s.close()
    np.testing.assert_array_equal(want[-2], want[-1])
