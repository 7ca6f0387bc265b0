"""Batched calls on a capturing stream (a caller's own graph): replayed with
other calls on the same context, eager work and synchronizations in between,
every replay gives what the call gives when it is made directly."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu


def _capture(call):
    import torch

    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    return graph


def test_captured_row_tables_keep_their_rows():
    import torch

    lengths = [[30000, 20, 40000], [5, 70000], [300, 300, 300, 1 << 20], [2048], [1 << 18, 17000]]
    xs = [[synth.lognormal_f32(n, 700 + 10 * t + k, 1.0) for k, n in enumerate(ls)] for t, ls in enumerate(lengths)]
    ins = [[torch.from_numpy(x).cuda() for x in rows] for rows in xs]
    outs = [[torch.zeros_like(x) for x in rows] for rows in ins]
    other = torch.rand(60000, device="cuda") + 0.5
    other_out = torch.empty_like(other)
    ctx = api.Context()
    ctx.batch_reserve(64, 1 << 22)
    graphs = [_capture(lambda o=o, i=i: api.normalize_rows(list(zip(o, i)), ctx=ctx)) for o, i in zip(outs, ins)]
    for turn in range(3):
        for rows in outs:
            for o in rows:
                o.fill_(-1.0)
        for graph in graphs:
            graph.replay()
            api.normalize_rows([(other_out[:50000], other[:50000]), (other_out[50000:], other[50000:])], ctx=ctx)
            if turn == 1:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        for rows, want in zip(outs, xs):
            for o, x in zip(rows, want):
                assert_f32_close(o.cpu().numpy(), oracle.normalize(x), what="replay %d, row of %d" % (turn, x.size))
    assert ctx.device_error() == L.NRM_OK
    del graphs
    ctx.close()


def test_captured_large_batch():
    """2^27 elements of capacity: a direct call replays the library's own graph."""
    import torch

    inp = torch.zeros(1 << 27, device="cuda")
    out = torch.empty_like(inp)
    offs = synth.ragged_offsets(np.array([700, 40000, 0, 1 << 20, 3000000, 256], np.int64))
    x = synth.lognormal_f32(int(offs[-1]), 720, 1.0)
    inp[:x.size] = torch.from_numpy(x).cuda()
    offs_d = torch.from_numpy(offs).cuda()
    ctx = api.Context()
    ctx.batch_reserve(64, 1 << 27)
    graph = _capture(lambda: api.normalize_batched(out, inp, offs_d, ctx=ctx))
    ref = oracle.normalize_batched(x, offs)
    for turn in range(3):
        out[:x.size] = -1.0
        graph.replay()
        assert_f32_close(out[:x.size].cpu().numpy(), ref, what="replay %d" % turn)
        out[:x.size] = -1.0
        api.normalize_batched(out, inp, offs_d, ctx=ctx)
        assert_f32_close(out[:x.size].cpu().numpy(), ref, what="direct %d" % turn)
    assert ctx.device_error() == L.NRM_OK
    del graph
    ctx.close()
