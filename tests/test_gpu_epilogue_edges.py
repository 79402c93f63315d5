"""Staged output of the expert GEMMs at the edges of its row groups, with rows behind the last one that have to stay
untouched: one expert of n rows, n around the multiples of 8, 16 and 32 rows that leave together (few work items, so
the device cuts it to tiles of one to four blocks of 32 rows in the tall class and of one block in the others), and 128
experts that fill whole rounds with uncut tiles, the last of them, of every height, ragged or full, at the end of the
buffer (test_schedule_entries.py holds the work lists to that)."""
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


# 128 experts, d = 1024, f = 256 or 768: 256 or 768 and 512 work items (class 5: 512 and 1024) if no expert is cut, which are
# whole rounds.  Loads by class and kind of stores: f, rows of all experts but the last, 32-row blocks of the last one.
E, D = 128, 1024
TALL = [32 * (5 + e % 5) - (0, 1, 13, 31)[e // 5 % 4] for e in range(E - 1)]
WHOLE_LOADS = {
    (1, "plain"): (256, TALL, (5, 6, 7, 8, 9)),
    (1, "device scope"): (768, [n if e % 2 else 1 + e % 32 for e, n in enumerate(TALL)], (5, 6, 7, 8, 9)),
    (0, "plain"): (256, [32 * (2 + e % 3) - (0, 5, 31)[e // 3 % 3] for e in range(E - 1)], (2, 3, 4)),
    (5, "plain"): (256, [64 - e % 40 for e in range(E - 1)], (1, 2)),
}
LAST = (0, 1, 13, 24, 31)  # rows missing from the last block


def experts(f):
    import torch
    g = torch.Generator().manual_seed(3)
    return [torch.empty(s, dtype=torch.bfloat16).normal_(0, a ** -0.5, generator=g) for s, a in
            (((E, D, f), D), ((E, D, f), D), ((E, f, D), f))]


@pytest.mark.parametrize("cls,stores", sorted(WHOLE_LOADS))
def test_last_rows_of_whole_tiles(cls, stores):
    import torch
    import paper_2605_19945_amd as moe
    f, rows, heights = WHOLE_LOADS[cls, stores]
    weights = experts(f)
    head, most = sum(rows), 32 * max(heights)
    ctx = moe.MoEContext(head + most, D, f, E, 1)
    ctx.moe_set_tile_class(cls)
    packed = ctx.moe_pack_weights(*[w.cuda() for w in weights])
    xp = wl.gaussian_bf16_bits(5, cls, (head + most, D), 1.0)
    off = np.concatenate([[0], np.cumsum(rows + [most])]).astype(np.int32)
    ref = orc.grouped_ffn(xp, off, *[gu.bits_of(w) for w in weights])
    x, first = gu.to_dev_bf16(xp), None
    for n in sorted({32 * h - less for h in heights for less in LAST}):
        print(f"class {cls}, {stores}, last expert of {n} rows", flush=True)
        off[E] = head + n
        y = torch.full((head + n + 32, D), 7.0, dtype=torch.bfloat16, device="cuda")
        ctx.moe_grouped_ffn(x[:head + n], gu.to_dev(off), head + n, packed, y=y[:head + n])
        torch.cuda.synchronize()
        gu.check_output(gu.f64_of_bf16(y[head:head + n]), ref[head:head + n], what=f"class {cls}, {stores}, last {n} rows")
        assert bool((y[head + n:] == 7.0).all()), f"rows past {n} were written"
        if first is None:
            first = y[:head].clone()
            gu.check_output(gu.f64_of_bf16(first), ref[:head], what=f"class {cls}, {stores}, all rows")
        assert torch.equal(y[:head], first)
    ctx.close()
