"""Large batches mostly of long rows, whose long rows get launches of their own:
every row has the bits that it has alone (in the persistent kernel), and the
oracle's value within the stated bounds."""
import numpy as np
import pytest

import oracle
from paper_2207_00257_amd import _lib as L
from paper_2207_00257_amd import api, synth
from parity_util import assert_f32_close

pytestmark = pytest.mark.gpu

# 2^26 elements, mean above 2^20: long rows (one whose last tile has one element), a resident row, short and empty ones
LENGTHS = [9000000, 1 << 20, (1 << 20) + 1, 20000000, 0, 300, (1 << 25) + 17, 40000, 4000000]


@pytest.mark.parametrize("kind", ["f32", "kahan", "bf16", "softmax", "table"])
def test_rows_have_the_bits_they_have_alone(kind):
    import torch

    rng = np.random.default_rng(91)
    offs = synth.ragged_offsets(np.array(LENGTHS, np.int64)) + 5
    total = int(offs[-1])
    assert total >= 1 << 26 and total // len(LENGTHS) > 1 << 20
    x = rng.random(total, dtype=np.float32) + np.float32(0.5)
    inp = torch.from_numpy(x).cuda()
    if kind == "bf16":
        inp = inp.to(torch.bfloat16)
    out, one = torch.zeros_like(inp), torch.zeros_like(inp)
    offs_d = torch.from_numpy(offs).cuda()
    accum = "kahan" if kind == "kahan" else "f32"
    lse, lse_one = torch.zeros(len(LENGTHS), device="cuda"), torch.zeros(len(LENGTHS), device="cuda")
    with_rows, alone = api.Context(), api.Context()

    def call(o, r0, r1, ctx, ls):
        b, e = int(offs[r0]), int(offs[r1])
        if kind == "table":
            rows = [(o[offs[r]:offs[r + 1]], inp[offs[r]:offs[r + 1]]) for r in range(r0, r1)]
            return api.normalize_rows(rows, ctx=ctx)
        # a row alone: its own slice as the arrays, so that the batch is no large one
        oo, ii, of = (o, inp, offs_d) if r1 - r0 > 1 else (o[b:e], inp[b:e], offs_d[r0:r1 + 1] - b)
        if kind == "softmax":
            return api.softmax_batched(oo, ii, of, lse=ls[r0:r1], ctx=ctx)
        return api.normalize_batched(oo, ii, of, accum=accum, ctx=ctx)

    for _ in range(2):
        call(out, 0, len(LENGTHS), with_rows, lse)
    for r, n in enumerate(LENGTHS):
        assert n < 1 << 26
        call(one, r, r + 1, alone, lse_one)
    assert with_rows.device_error() == L.NRM_OK and alone.device_error() == L.NRM_OK
    same = (out.view(torch.int16) == one.view(torch.int16)) if kind == "bf16" else (out.view(torch.int32) == one.view(torch.int32))
    assert bool(same.all())
    if kind == "softmax":
        assert bool((lse.view(torch.int32) == lse_one.view(torch.int32)).all())
    elif kind != "bf16":
        assert_f32_close(out[5:].cpu().numpy(), oracle.normalize_batched(x, offs)[5:], what=kind)
    with_rows.close()
    alone.close()
