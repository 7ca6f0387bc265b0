"""The captured launch sequence of large batches (at least 2^27 elements of
capacity): its first launch's arguments and grid are set anew for every replay."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu


def test_replays_with_other_rows_and_eager_work_between():
    """Seven batches of other row counts, lengths and offsets through one
    context, the replays' buffers and graphs used in turn, with eager library
    calls and synchronizations between some of them: each result is that of
    the same batch launched directly, bit for bit, and the oracle's within the
    stated bound. The arrays have 2^27 elements, of which the rows cover a part."""
    import torch

    inp = torch.zeros(1 << 27, device="cuda")
    gctx, dctx = api.Context(), api.Context()
    gctx.set_batch_params(graph=1)
    dctx.set_batch_params(graph=0)
    for k, (rows, hi) in enumerate(((3000, 3000), (20, 1 << 20), (9000, 300), (1, 7), (400, 40000), (3, 1 << 21), (5000, 900))):
        lengths = synth.loguniform_lengths(rows, 600 + k, 1, hi)
        offs = synth.ragged_offsets(lengths) + 32 * k
        x = synth.lognormal_f32(int(offs[-1]), 620 + k, 1.0)
        inp[:x.size] = torch.from_numpy(x).cuda()
        o = torch.from_numpy(offs).cuda()
        outs = [torch.empty_like(inp) for _ in range(2)]
        for t, c in zip(outs, (gctx, dctx)):
            t[:x.size] = -1.0
            api.normalize_batched(t, inp, o, ctx=c)
            if k % 2:
                small = torch.rand(1000, device="cuda")
                api.normalize(small, small)
                torch.cuda.synchronize()
        g, d = (t[:x.size].cpu().numpy() for t in outs)
        assert np.array_equal(g.view(np.uint32), d.view(np.uint32)), k
        b = int(offs[0])
        assert_f32_close(g[b:], oracle.normalize_batched(x, offs)[b:], what="replay %d" % k)
    assert gctx.device_error() == L.NRM_OK
    gctx.close()
    dctx.close()
