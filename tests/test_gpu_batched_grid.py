"""A batch with more blocks than one row of the grid of its first launch takes
(2^20): 2^21 + 5 rows, two per block, nearly all of them empty, the others at
the start, on both sides of the grid's second row and at the end."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_within_ulp, bf16_bits_to_f64, ulp_bf16

pytestmark = pytest.mark.gpu

ROWS = (1 << 21) + 5
HALF = (1 << 20) + 4  # rows of the first row of the grid: half of the 2^20 + 3 blocks, rounded up


@pytest.mark.parametrize("graph", [0, 1])
def test_rows_in_the_second_row_of_the_grid(graph):
    import torch

    lengths = np.zeros(ROWS, np.int64)
    at = {0: 7, 1: 300, HALF - 2: 2049, HALF - 1: 40000, HALF: 256, HALF + 1: (1 << 20) + 5, HALF + 2: 90000,
          ROWS - 2: 3000, ROWS - 1: 2048}
    for r, n in at.items():
        lengths[r] = n
    offs = synth.ragged_offsets(lengths)
    total = int(offs[-1])
    bits = synth.f32_to_bf16_bits(synth.lognormal_f32(total, 31, 1.0))
    # two rows per block are for a mean of 4096 and more: the rows cover a small part of the array
    buf = torch.empty(4096 * ROWS, dtype=torch.bfloat16, device="cuda")
    buf[:total] = torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)
    ctx = api.Context()
    ctx.set_batch_params(graph=graph)
    api.normalize_batched(buf, buf, torch.from_numpy(offs).cuda(), ctx=ctx)
    assert ctx.device_error() == L.NRM_OK
    ctx.close()
    got = bf16_bits_to_f64(buf[:total].view(torch.int16).cpu().numpy().view(np.uint16))
    del buf
    torch.cuda.empty_cache()
    assert_within_ulp(got, oracle.normalize_batched(bits, offs, "bf16"), ulp_bf16, what="graph=%d" % graph)
