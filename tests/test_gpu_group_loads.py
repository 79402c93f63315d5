"""Expert FFN over rows per expert that mix heavy experts, experts of several row tiles and light ones, and over many
experts whose row tiles stay whole up to the tallest one, at the numbers of K steps around the length of the pipeline: all
rows against the oracle."""
import numpy as np
import pytest

from oracle import moe_oracle as orc

import gpu_util as gu

pytestmark = pytest.mark.gpu

LOADS = {
    "one_to_nine_blocks": [1, 33, 65, 128, 129, 161, 224, 225, 287, 288, 289, 40],
    "heavy_and_few_light": [300, 0, 5, 96, 97, 31, 700, 2],        # fewer than eight light tiles to deal
    "light_only": [1, 0, 20, 33, 64, 90, 7, 3, 0, 12, 32],         # some of two and three blocks
    "one_block_each": [1, 32, 17, 0, 5, 30, 31, 2, 9],             # one stretch per XCD
    "eight_row_tiles_and_more": [2500, 4, 40, 600],                # two row ranges
}


def _bits(rng, *shape, std=1.0):
    a = rng.standard_normal(shape, dtype=np.float32) * std
    u = a.view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)


# Few work items make the device cut tiles to four blocks and less; 256 experts of five to nine blocks fill whole rounds
# with uncut ones (test_schedule_entries.py holds the work lists to that).  Last blocks of 1, 19, 31 and 32 rows.
TALL_ROWS = [32 * (5 + e % 5) - (0, 1, 13, 31)[e // 5 % 4] for e in range(256)]
TALL_WIDTHS = [(64, 64), (128, 192), (192, 320), (256, 128), (320, 256)]  # one to five K steps in either GEMM


def _against_the_oracle(rows, d, f, cls, what):
    import torch
    import paper_2605_19945_amd as moe
    E, n = len(rows), sum(rows)
    print(f"{what} d={d} f={f} cls={cls}", flush=True)
    rng = np.random.default_rng(d + 7 * f + len(rows))
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    xp = _bits(rng, n, d)
    W1, W3, W2 = _bits(rng, E, d, f, std=d ** -0.5), _bits(rng, E, d, f, std=d ** -0.5), _bits(rng, E, f, d, std=f ** -0.5)
    ctx = moe.MoEContext(n, d, f, E, 1)
    ctx.moe_set_tile_class(cls)
    packed = ctx.moe_pack_weights(gu.to_dev_bf16(W1), gu.to_dev_bf16(W3), gu.to_dev_bf16(W2))
    y = torch.full((n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ctx.moe_grouped_ffn(gu.to_dev_bf16(xp), gu.to_dev(off), n, packed, y=y)
    torch.cuda.synchronize()
    ctx.close()
    # one rounding of the intermediate and one of the result, bounded as in the other parity tests; a row that no work
    # item holds stays NaN
    gu.check_output(gu.f64_of_bf16(y), orc.grouped_ffn(xp, off, W1, W3, W2), what=f"{what} d={d} f={f} cls={cls}")


@pytest.mark.parametrize("cls", [-1, 0, 1, 5])
@pytest.mark.parametrize("d,f", [(64, 64), (128, 192), (192, 320), (256, 448), (320, 576), (704, 128)])
@pytest.mark.parametrize("load", sorted(LOADS))
def test_rows_against_the_oracle(load, d, f, cls):
    _against_the_oracle(LOADS[load], d, f, cls, load)


@pytest.mark.parametrize("d,f", TALL_WIDTHS)
def test_tall_tiles_against_the_oracle(d, f):
    _against_the_oracle(TALL_ROWS, d, f, 1, "tall")
