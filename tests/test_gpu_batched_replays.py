"""Replays of the library's own graph (batches of 2^27 elements and more, not
mostly of long rows) of the kinds that test_gpu_batched_graph.py has not:
compensated sums and row tables, each with other contents per call and eager
work in between; the results are those of direct launches, bit for bit, and the
oracle's within the stated bounds."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu


def _between(k):
    import torch

    if k % 2:
        small = torch.rand(1000, device="cuda")
        api.normalize(small, small)
        torch.cuda.synchronize()


def test_compensated_replays():
    import torch

    inp = torch.zeros(1 << 27, device="cuda")
    ctxs = [api.Context(), api.Context()]
    ctxs[1].set_batch_params(graph=0)
    outs = [torch.empty_like(inp) for _ in ctxs]
    for k, (rows, hi) in enumerate(((3000, 3000), (800, 40000), (9000, 300), (600, 1 << 18), (2000, 20000), (5000, 900))):
        offs = synth.ragged_offsets(synth.loguniform_lengths(rows, 640 + k, 1, hi)) + 32 * k
        x = synth.lognormal_f32(int(offs[-1]), 660 + k, 2.0)
        inp[:x.size] = torch.from_numpy(x).cuda()
        offs_d = torch.from_numpy(offs).cuda()
        for o, c in zip(outs, ctxs):
            o[:x.size] = -1.0
            api.normalize_batched(o, inp, offs_d, accum="kahan", ctx=c)
            _between(k)
        g, d = (o[:x.size].cpu().numpy() for o in outs)
        assert np.array_equal(g.view(np.uint32), d.view(np.uint32)), k
        b = int(offs[0])
        assert_f32_close(g[b:], oracle.normalize_batched(x, offs)[b:], what="replay %d" % k)
    for c in ctxs:
        assert c.device_error() == L.NRM_OK
        c.close()


def test_row_table_replays():
    """520 rows of 2^27 elements and more together: mean below a quarter of the
    resident limit. Rows of mixed dtypes, in other places and lengths per call."""
    import torch

    base, rows = (1 << 27) // 520 + 1, 520
    buf = torch.empty(rows * (base + 700), device="cuda").uniform_(0.5, 1.5)
    half = buf.to(torch.bfloat16)
    ctxs = [api.Context(), api.Context()]
    ctxs[1].set_batch_params(graph=0)
    outs = [torch.empty_like(buf) for _ in ctxs]
    for k in range(5):
        rng = np.random.default_rng(680 + k)
        lengths = base + rng.permutation(rows) - rows // 2 + 400
        lengths[:4] = [base + 650, base + 650, 700, base + 650]
        lengths[4:20] += base // 16  # (makes up for the short row)
        offs = synth.ragged_offsets(lengths.astype(np.int64))
        assert (1 << 27) <= offs[-1] <= buf.numel() and offs[-1] // rows < 1 << 18
        for o, c in zip(outs, ctxs):
            o.fill_(-1.0)
            pairs = [(o[offs[r]:offs[r + 1]], (half if r % 3 == 1 else buf)[offs[r]:offs[r + 1]]) for r in range(rows)]
            api.normalize_rows(pairs, ctx=c)
            _between(k)
        assert bool((outs[0].view(torch.int32) == outs[1].view(torch.int32)).all()), k
        for r in (0, 1, 2, 3, 100, rows - 1):
            src = (half if r % 3 == 1 else buf)[offs[r]:offs[r + 1]].float().cpu().numpy()
            assert_f32_close(outs[0][offs[r]:offs[r + 1]].cpu().numpy(), oracle.normalize(src), what="replay %d row %d" % (k, r))
    for c in ctxs:
        assert c.device_error() == L.NRM_OK
        c.close()
