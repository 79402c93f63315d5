"""Staged output of the expert GEMMs at the edges of its row groups: one expert of n rows, n around the multiples of 8, 16
and 32 rows that leave together, of full and ragged tiles of every height, stored through the L2 (up to one tall tile) and
not; rows behind the last one stay untouched."""
import numpy as np
import pytest

import gpu_util as gu
import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cls,rows", [(0, (1, 7, 33, 64, 65, 96, 127, 128, 129)), (5, (1, 31, 32, 33, 63, 64, 65)),
                                      (1, (1, 15, 32, 47, 64, 97, 160, 191, 224, 255, 256, 257, 280, 287, 288, 289, 575, 577))])
def test_rows_at_the_edges_of_the_groups(cls, rows):
    import torch
    import paper_2605_19945_amd as moe
    d, f = 320, 192  # neither a multiple of the weight-row tile
    W1, W3, W2 = wl.expert_weights(5, 1, d, f, 0.08)
    ctx = moe.MoEContext(max(rows), d, f, 1, 1)
    packed = ctx.moe_pack_weights(gu.to_dev_bf16(W1), gu.to_dev_bf16(W3), gu.to_dev_bf16(W2))
    ctx.moe_set_tile_class(cls)
    xp = wl.gaussian_bf16_bits(5, 9, (max(rows), d), 1.0)
    ref = orc.grouped_ffn(xp, np.array([0, max(rows)], np.int32), W1, W3, W2)
    x = gu.to_dev_bf16(xp)
    for n in rows:
        print(f"class {cls}, {n} rows", flush=True)
        y = torch.full((max(rows) + 32, d), 7.0, dtype=torch.bfloat16, device="cuda")
        ctx.moe_grouped_ffn(x[:n], torch.tensor([0, n], dtype=torch.int32, device="cuda"), n, packed, y=y[:n])
        torch.cuda.synchronize()
        gu.check_output(gu.f64_of_bf16(y[:n]), ref[:n], what=f"class {cls}, {n} rows")
        assert bool((y[n:] == 7.0).all()), f"rows past {n} were written"
    ctx.close()
