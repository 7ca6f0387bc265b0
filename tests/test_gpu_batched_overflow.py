"""Rows that need more list entries than the workspace holds for the capacity
(offsets that go back and forth make every other row valid and all of those the
same slice): the rows that do not fit are skipped and the cause is named, those
that fit are right."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pairs,capacity,params", [
    (80000, 1000, 80000, {}), ((1 << 20) + 5, 100, (1 << 20) + 5, {}), (80000, 1000, 80000, dict(resident_segments=0)),
    ((1 << 20) + 5, 100, (1 << 20) + 5, dict(resident_segments=0)), (1 << 21, 256, 1 << 27, {})])  # the last: long rows apart
def test_rows_that_do_not_fit_are_named_and_the_others_right(n, pairs, capacity, params):
    import torch

    x = synth.lognormal_f32(n, 5, 1.0)
    inp = torch.zeros(capacity, device="cuda")
    inp[:n] = torch.from_numpy(x).cuda()
    out = torch.zeros_like(inp)
    ctx = api.Context()
    ctx.set_batch_params(**params)
    offs = np.tile(np.array([0, n], np.int64), pairs)
    api.normalize_batched(out, inp, torch.from_numpy(offs).cuda(), ctx=ctx)
    assert ctx.device_error() == L.NRM_EDEVICE
    assert b"batch larger than the workspace" in L.lib().nrm_last_error()
    assert_f32_close(out[:n].cpu().numpy(), oracle.normalize(x), what="a row that fits")
    # offsets that go back, without more entries than fit: another cause alone
    api.normalize_batched(out, inp, torch.from_numpy(offs[:4].copy()).cuda(), ctx=ctx)
    assert ctx.device_error() == L.NRM_EDEVICE
    assert b"workspace" not in L.lib().nrm_last_error()
    ctx.close()
