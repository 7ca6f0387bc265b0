"""The plain call's one-launch form with fewer blocks than segments, as when not
all of a launch's blocks can run: the running ones take the other segments
over. The internal launch is called for it (the entry points always launch one
block per segment)."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu

LAUNCH = "_ZN3nrm21launch_plain_residentEPKviPviliRKNS_15PlainResidentWsEP12ihipStream_t"


class Ws(ctypes.Structure):
    _fields_ = [("slots", ctypes.c_void_p), ("arrivals", ctypes.c_void_p), ("call", ctypes.c_void_p),
                ("sum_out", ctypes.c_void_p), ("blocks", ctypes.c_uint)]


def _launcher():
    fn = getattr(L.lib(), LAUNCH)
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_int,
                   ctypes.POINTER(Ws), ctypes.c_void_p]
    return fn


@pytest.mark.parametrize("accum", ["f32", "kahan"])
@pytest.mark.parametrize("n", [4096, 4097, 3 * 4096 + 5, 1 << 18, (1 << 18) + 1, 1 << 19])
def test_fewer_blocks_than_segments(n, accum):
    """The same bits as with a block per segment, out of place and in place,
    calls of different block counts one after the other on one workspace."""
    import torch

    launch = _launcher()
    mem = torch.zeros(512, dtype=torch.int64, device="cuda")
    base = mem.data_ptr()
    x = synth.lognormal_f32(n + 1, 800, 1.0)
    buf = torch.from_numpy(x).cuda()
    inp = buf[1:]
    want = torch.empty_like(inp)
    ctx = api.Context()
    api.normalize(want, inp, accum=accum, ctx=ctx)
    assert_f32_close(want.cpu().numpy(), oracle.normalize(x[1:]), what="n=%d" % n)
    acc = {"f32": L.NRM_ACC_F32, "kahan": L.NRM_ACC_KAHAN}[accum]
    stream = torch.cuda.current_stream().cuda_stream
    for blocks in (1, 0, 2, 5, 63, 0, 1):
        ws = Ws(base + 512, base + 8, base, base + 256, blocks)
        for in_place in (False, True):
            work = buf.clone()[1:]
            out = work if in_place else torch.zeros(n + 1, device="cuda")[1:]
            torch.cuda.synchronize()
            print("n=%d %s blocks=%d in_place=%d" % (n, accum, blocks, in_place), flush=True)
            assert launch(work.data_ptr(), L.NRM_F32, out.data_ptr(), L.NRM_F32, n, acc, ctypes.byref(ws), stream) == 0
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.cpu().numpy().view(np.uint32)), (blocks, in_place)
    assert mem[1].item() == 0  # every block has arrived
    ctx.close()
