"""Batches at the sizes where the batched path changes how it is cut up: rows
per block of the rows' kernel (1, 2, 4, 8, 32), rows run on 16 lanes, on a
wavefront, by a block, listed as segments or as tiles, each at the limits of
its range, at whole-line and other starts; every row against the FP64 oracle
within the stated bounds (tests/parity_util.py)."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close, assert_within_ulp, bf16_bits_to_f64, ulp_bf16

pytestmark = pytest.mark.gpu

EDGES = [1, 15, 16, 17, 255, 256, 257, 2047, 2048, 2049, (1 << 14) - 1, 1 << 14, (1 << 14) + 1, 3 << 14]
# (rows, lengths to draw from): the mean length and the row count pick the cut
CUTS = {
    "one_row_per_block": (400, EDGES + [1 << 20, (1 << 20) + 1, (1 << 20) + 40000]),
    "listed_with_long_rows": (700, [100, 300, 2049, 1 << 14, (1 << 14) + 1, 40000, 90000]),
    "two_rows_per_block": (1500, [64, 2048, 2049, 8000, 1 << 14]),
    "four_rows_per_block": (3000, [17, 256, 1500, 2048, 2049, 4096]),
    "eight_rows_per_block": (5000, [1, 250, 256, 257, 1000, 2048]),
    "thirty_two_rows_per_block": (9000, [0, 1, 3, 64, 250, 256, 257, 300, 2049]),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 5])
@pytest.mark.parametrize("cut", list(CUTS))
def test_rows_at_the_limits_of_each_cut(cut, shift, dtype):
    import torch

    rows, choices = CUTS[cut]
    rng = np.random.default_rng(7 + rows)
    lengths = rng.choice(np.array(choices, np.int64), rows)
    offs = synth.ragged_offsets(lengths) + shift
    x = synth.lognormal_f32(int(offs[-1]), 11 + rows, 1.0)
    host = x if dtype == "f32" else synth.f32_to_bf16_bits(x)
    inp = torch.from_numpy(host if dtype == "f32" else host.view(np.int16)).cuda()
    if dtype == "bf16":
        inp = inp.view(torch.bfloat16)
    out = torch.zeros_like(inp)
    ctx = api.Context()
    api.normalize_batched(out, inp, torch.from_numpy(offs).cuda(), ctx=ctx)
    assert ctx.device_error() == L.NRM_OK
    ctx.close()
    ref = oracle.normalize_batched(host, offs, dtype)[shift:]
    if dtype == "f32":
        assert_f32_close(out.cpu().numpy()[shift:], ref, what=cut)
    else:
        got = bf16_bits_to_f64(out.view(torch.int16).cpu().numpy().view(np.uint16))[shift:]
        assert_within_ulp(got, ref, ulp_bf16, what=cut)


def test_overlapping_rows_beyond_the_workspace_are_flagged():
    """Offsets that go back and forth make every other row valid and all of
    them the same slice: their segments exceed what the workspace holds for
    the capacity. The call ends, is flagged, and the next one is whole."""
    import torch

    n, pairs = 40000, 1000
    x = synth.lognormal_f32(n, 5, 1.0)
    inp = torch.from_numpy(x).cuda()
    out = torch.zeros_like(inp)
    ctx = api.Context()
    offs = np.tile(np.array([0, n], np.int64), pairs)
    api.normalize_batched(out, inp, torch.from_numpy(offs).cuda(), ctx=ctx)
    assert ctx.device_error() == L.NRM_EDEVICE
    api.normalize_batched(out, inp, torch.from_numpy(offs[:2].copy()).cuda(), ctx=ctx)
    assert ctx.device_error() == L.NRM_OK
    assert_f32_close(out.cpu().numpy(), oracle.normalize(x), what="after the flagged call")
    ctx.close()
