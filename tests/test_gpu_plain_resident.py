"""The plain call's one-launch form at the sizes where its segments change
(2^12 elements up to 2^18, 2^14 above, the two kernels beyond 2^20, compensated
beyond 2^19), with the library's own choice, against the FP64 oracle within the
stated bounds; and several such calls running at once on streams of their own."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("accum", ["f32", "kahan"])
@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1, (17 << 14) + 1, (1 << 19) - 3, 1 << 19, (1 << 19) + 1,
                               (1 << 20) - 1, 1 << 20, (1 << 20) + 1])
def test_sizes_where_the_form_changes(n, accum):
    import torch

    x = synth.lognormal_f32(n + 3, 400, 1.0)
    buf = torch.from_numpy(x).cuda()
    ctx = api.Context()
    for off in (0, 3):  # a start on a line, and one that is not
        inp = buf[off:off + n]
        out = torch.zeros(n + 3, device="cuda")[off:off + n]
        for _ in range(2):
            api.normalize(out, inp, accum=accum, ctx=ctx)
        assert_f32_close(out.cpu().numpy(), oracle.normalize(x[off:off + n]), what="n=%d off=%d %s" % (n, off, accum))
    assert ctx.device_error() == L.NRM_OK
    ctx.close()


def test_calls_at_once_on_many_streams():
    """Sixteen contexts, each on a stream of its own, twenty calls each with
    nothing waiting in between: their blocks share the device, every call ends
    with its own sum and no wait gives up."""
    import torch

    sizes = [(1 << 20) - 64 * k for k in range(16)]
    xs = [synth.lognormal_f32(n, 420 + k, 1.0) for k, n in enumerate(sizes)]
    ins = [torch.from_numpy(x).cuda() for x in xs]
    outs = [torch.zeros_like(t) for t in ins]
    ctxs = [api.Context() for _ in sizes]
    streams = [torch.cuda.Stream() for _ in sizes]
    torch.cuda.synchronize()
    for _ in range(20):
        for c, s, o, t in zip(ctxs, streams, outs, ins):
            api.normalize(o, t, ctx=c, stream=s.cuda_stream)
    torch.cuda.synchronize()
    for c, o, x in zip(ctxs, outs, xs):
        assert c.device_error() == L.NRM_OK
        assert_f32_close(o.cpu().numpy(), oracle.normalize(x), what="n=%d" % x.size)
        c.close()
