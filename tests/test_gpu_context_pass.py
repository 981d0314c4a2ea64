"""The context pass on a kept handle: batches of one shape after another replay captured launches, a change of shape
rebuilds them.  Every forecast must equal, to the bit, the one a fresh handle makes of the same series."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2511_18191_amd as tsd
import synth
from harness import TOL, Case, lockstep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["cfg1", "mini2", "mini5"])
def test_forecasts_of_a_kept_handle_equal_a_fresh_handles(name):
    case = Case(name, B=6)
    c = case.cfg
    P, N, H = c.patch, c.n_ctx, c.horizon
    sess = case.session()
    rng = np.random.default_rng(5)
    # (series, context patches, horizon): the same shape three times (launch by launch, captured, replayed), then other
    # batch sizes, contexts and horizons, and the first shape again
    for B, n, h in [(6, N, H)] * 3 + [(4, N, H)] * 2 + [(4, N - 1, H), (4, N - 1, H - P)] + [(6, N, H)] * 2:
        ctx = np.roll(case.context[:B, :n * P], int(rng.integers(1, n * P)), axis=1)   # other inputs every time
        sess.prefill(ctx, n, h)
        sess.run_rounds()
        got = sess.get_forecast().cpu().numpy()
        fresh = case.session()
        fresh.prefill(ctx, n, h)
        fresh.run_rounds()
        np.testing.assert_array_equal(got, fresh.get_forecast().cpu().numpy(), err_msg=f"{B} series of {n} patches, {h} steps")
        fresh.close()
    sess.close()


def test_eager_prefill_after_a_captured_one_uploads_the_page_table():
    """A prefill the caller captures runs at its replays only: the next eager one must not take its page table for uploaded."""
    case = Case("mini2", B=4)
    c = case.cfg
    sess = case.session()
    sess.prefill(case.context[:2], c.n_ctx, c.horizon)
    series = sess._to_dev(case.context, torch.float32)
    sess.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=sess.stream, capture_error_mode="thread_local"):
        rc = tsd.lib().tsd_prefill(sess.h, series.data_ptr(), 4, c.n_ctx, c.horizon, sess.stream.cuda_stream)
    assert rc == 0
    fresh = case.session()
    for s in (sess, fresh):
        s.prefill(case.context, c.n_ctx, c.horizon)
        s.run_rounds()
    np.testing.assert_array_equal(sess.get_forecast().cpu().numpy(), fresh.get_forecast().cpu().numpy())
    sess.close()
    fresh.close()


@pytest.mark.parametrize("B,N", [(1, 17), (3, 18), (3, 34), (5, 50), (9, 82)])
def test_context_of_several_query_tiles(B, N):
    """Contexts of 16, 17, 33, 49 and 81 rows: one to six 16-query tiles per (series, head), whole and ragged last ones,
    numbers of (series, head) that are and are not multiples of eight, against the oracle."""
    case = Case("mini2", B=B, context=N * synth.CONFIGS["mini2"].patch)
    sess = case.session()
    rep = lockstep(case, sess, max_rounds=1)
    assert rep["max_rel_X"] <= TOL["bf16"] and rep["max_rel_mu_p"] <= TOL["bf16"], rep
    sess.close()


@pytest.mark.parametrize("name,B", [("cfg1", 6), ("mini2", 2), ("mini2", 6), ("mini2", 40), ("mini5", 6),
                                    ("mini3", 20), ("mini3", 1200), ("mini3", 1240)])   # (rounds on 64-, 128- and 256-row tiles)
def test_smaller_arenas(name, B):
    """Every arena between the least and the full size decodes, to the bit as the full one does: the context in more passes, without the
    resident kernel, without the table of row positions."""
    case = Case(name, B=B)
    c = case.cfg
    L, n = tsd.lib(), C.c_size_t()
    sess = case.session()
    full = sess.arena_bytes
    base = (sess.arena.data_ptr() + 255) & ~255

    def arena(size):
        sess.close()
        h = C.c_void_p()
        rc = L.tsd_create(C.byref(sess.cfg), base, size, C.byref(h))
        if rc:
            return False
        sess.h = h
        for which, m, w in ((tsd.TSD_TARGET, c.target, case.wt), (tsd.TSD_DRAFT, c.draft, case.wd)):
            sess.load_weights(which, synth.flatten_weights(m, c.patch, w))
        return True

    def decode():
        sess.prefill(case.context, c.n_ctx, c.horizon)
        sess.run_rounds()
        out = [sess.get_forecast().cpu().numpy()]
        sess.reset_decode()
        for _ in range(c.T):
            sess.target_step()
        return out + [sess.get_forecast().cpu().numpy()]

    want = decode()
    resident = sess.resident_passes()
    lo, hi = 0, full                      # refused, accepted
    while hi - lo > 256:
        mid = (lo + hi) // 512 * 256
        if arena(mid):
            hi = mid
        else:
            lo = mid
    least, seen = hi, set()
    # the least; with row positions; with the resident kernel too; a few rows more; half way; all but the last rows
    for size in (least, least + 16384, least + 65536, (least + full) // 2, full - 256, full):
        assert arena(min(size, full))
        for a, b in zip(decode(), want):
            np.testing.assert_array_equal(a, b, err_msg=f"{size} of {least} .. {full} bytes")
        seen.add(sess.resident_passes() > 0)
    assert seen == ({False, True} if resident else {False})
    sess.close()
