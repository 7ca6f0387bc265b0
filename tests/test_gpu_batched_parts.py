"""Long rows with the longest tiles that the parameters take: a tile of more
than 2^19 elements is summed in parts. Every row against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("accum", ["f32", "kahan"])
@pytest.mark.parametrize("tile_log2", [19, 20, 22])
def test_tiles_of_several_parts(tile_log2, accum):
    import torch

    lengths = np.array([(1 << 20) + 1, (1 << 22) + (1 << 19) + 5, 300, (1 << 21) + 3], np.int64)
    offs = synth.ragged_offsets(lengths)
    x = synth.lognormal_f32(int(offs[-1]), 51, 1.0)
    inp = torch.from_numpy(x).cuda()
    out = torch.empty_like(inp)
    ctx = api.Context()
    ctx.set_batch_params(tile_log2=tile_log2, block=1024, unroll=8)
    api.normalize_batched(out, inp, torch.from_numpy(offs).cuda(), accum=accum, ctx=ctx)
    assert ctx.device_error() == L.NRM_OK
    ctx.close()
    assert_f32_close(out.cpu().numpy(), oracle.normalize_batched(x, offs), what="tile_log2=%d %s" % (tile_log2, accum))
