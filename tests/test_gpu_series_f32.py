"""Small fp32 models run a series per workgroup (series_f32.hip): bit for bit the kernels it replaces, which the same handle takes under a
measurement, over the sizes where its indexing changes: 1 to 17 rows per pass, contexts of one and several blocks of rows, every
width and head size, patches that leave blocks and k-runs partly filled, pages of one token, and more series than fit the grid's first turn."""
import numpy as np
import pytest

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
