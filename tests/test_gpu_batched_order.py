"""Batches whose listed segments are ordered over several rounds of blocks, and
with more blocks than are ordered: every row against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu

# (rows, lengths, blocks of the first launch): 1, 4, 2 and 2 rows per block
BATCHES = {"1_round": (512, [5, 17000, 40000], 512), "2_rounds": (4096, [0, 0, 300, 300, 3000, 17000], 1024),
           "4_rounds": (4095, [10, 3000, 3000, 17000, 40000], 2048), "unordered": (4098, [10, 3000, 3000, 17000, 40000], 2049)}


@pytest.mark.parametrize("name", list(BATCHES))
def test_listed_rows_in_any_number_of_rounds(name):
    import torch

    rows, choices, blocks = BATCHES[name]
    rng = np.random.default_rng(rows)
    lengths = rng.choice(np.array(choices, np.int64), rows)
    per_block = {512: 1, 1024: 4, 2048: 2, 2049: 2}[blocks]
    mean = int(lengths.sum()) // rows
    assert (mean >= 4096) == (per_block == 2) or per_block == 1
    assert -(-rows // per_block) == blocks
    offs = synth.ragged_offsets(lengths)
    x = synth.lognormal_f32(int(offs[-1]), 61, 1.0)
    inp = torch.from_numpy(x).cuda()
    out = torch.empty_like(inp)
    ctx = api.Context()
    for _ in range(3):
        out.fill_(-1.0)
        api.normalize_batched(out, inp, torch.from_numpy(offs).cuda(), ctx=ctx)
        assert ctx.device_error() == L.NRM_OK
    ctx.close()
    assert_f32_close(out.cpu().numpy(), oracle.normalize_batched(x, offs), what=name)
