"""Work of the caller's stream beside the library's."""
import numpy as np
import pytest
import torch

from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [False, True])
def test_a_forecast_waits_for_the_readers_of_its_memory(side):
    """A freed forecast that a kernel of the caller's stream has still to read: the next one gets the same memory and must not be
    written before."""
    case = Case("cfg1", B=6)
    c = case.cfg
    sess = case.session()
    sess.prefill(case.context, c.n_ctx, c.horizon)
    sess.run_rounds()
    with torch.cuda.stream(torch.cuda.Stream() if side else torch.cuda.current_stream()):
        old = sess.get_forecast()
        want, read, at = old.cpu().numpy(), torch.zeros_like(old), old.data_ptr()
        sess.reset_decode()
        sess.target_step()
        torch.cuda._sleep(50_000_000)
        torch.add(old, 0.0, out=read)
        del old
        new = sess.get_forecast()
        assert new.data_ptr() == at  # (torch hands the block out again: what the wait is for)
        np.testing.assert_array_equal(read.cpu().numpy(), want)
        assert (new.cpu().numpy() != want).any()
    sess.close()
