"""Sums over the slabs of a split reduction (router top-k, combine) at every number of slabs, and work lists of very
unequal lengths: layer output against the staged calls bit for bit, routing against fp64 logits."""
import pytest

import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _layer_and_staged(inp):
    import torch
    import paper_2605_19945_amd as moe
    s = inp.shape
    ctx = moe.MoEContext(max(1, s.T), s.d, s.f, s.E, s.k, s.e_lo, s.E_local, 0)
    x, rp = gu.to_dev_bf16(inp.x), ctx.moe_pack_router(gu.to_dev(inp.Wg))
    packed = ctx.moe_pack_weights(gu.to_dev_bf16(inp.W1), gu.to_dev_bf16(inp.W3), gu.to_dev_bf16(inp.W2))
    out = ctx.moe_layer_forward(x, rp, None, packed)
    idx, w, _ = ctx.moe_route(x, rp)
    xp, offsets, row_of, _ = ctx.moe_permute(x, idx)
    y = ctx.moe_grouped_ffn(xp, offsets, ctx.rows_capacity(s.T), packed)
    staged = ctx.moe_combine(y, row_of, w)
    torch.cuda.synchronize()
    ctx.close()
    return out, staged


# f / 64 K steps: 2, 3, 5, 7 and 8 ranges of at least 16 K steps divide them; 16 and 31 cannot be split.  With d = 64 and
# f = 4096 the first work list is 128 times the second, with d = 4096 and f = 64 a sixteenth of it.
@pytest.mark.parametrize("T,d,f", [(1, 128, 2048), (3, 128, 3072), (1, 192, 5120), (2, 128, 7168), (5, 128, 8192),
                                   (1, 128, 1024), (1, 128, 1984), (700, 64, 4096), (700, 4096, 64)])
def test_layer_equals_staged_calls(T, d, f):
    print(f"T={T} d={d} f={f}", flush=True)
    out, staged = _layer_and_staged(wl.custom("split_sums", T, d, f, 4, 2, seed=T + f, wg_std=0.05, w_std=0.03))
    import torch
    assert torch.equal(out.view(torch.int16), staged.view(torch.int16))


# K steps of 64: d = 512 and 448 are not split, 1024 in 2, 2560 in 5, 3584 in 7, 4096 in 8 slabs at these T
@pytest.mark.parametrize("d", [448, 512, 1024, 2560, 3584, 4096])
@pytest.mark.parametrize("E,T", [(32, 1), (33, 5), (64, 129), (100, 77), (255, 3), (256, 300)])
def test_router_sums_every_slab_once(d, E, T):
    import torch
    import paper_2605_19945_amd as moe
    print(f"d={d} E={E} T={T}", flush=True)
    k = 8
    g = torch.Generator().manual_seed(d + E + T)
    x = torch.randn(T, d, generator=g).to(torch.bfloat16)
    Wg, bias = torch.randn(d, E, generator=g) / d ** 0.5, 0.5 * torch.randn(E, generator=g)
    ctx = moe.MoEContext(T, d, 64, E, k)
    idx, w, counts = ctx.moe_route(x.cuda(), ctx.moe_pack_router(Wg.cuda()), bias.cuda())
    torch.cuda.synchronize()
    idx, w = idx.cpu().long(), w.cpu()
    assert torch.equal(counts.cpu().long(), torch.bincount(idx.reshape(-1), minlength=E))
    logits = x.double() @ Wg.double() + bias.double()
    top = logits.topk(k + 1, dim=1)
    # Two logits that are each off by less than 1e-4 (see below) keep their order if they are 2e-4 apart.  The eight
    # gaps of a token average 0.05 or more here, so one token in 30 at most has a smaller one: nearly all of many
    # tokens are compared, while a single token may happen not to be.
    clear = (top.values[:, :-1] - top.values[:, 1:]).min(dim=1).values > 2e-4
    assert T < 64 or clear.sum() > 0.9 * T
    assert torch.equal(idx[clear], top.indices[clear, :k])
    # The router matrix is kept to 2^-18 relative and d products are added in fp32: with unit-variance logits the
    # error of a logit stays below 1e-4, and a gate weight moves by at most twice that, relatively.
    ref = torch.softmax(logits.gather(1, idx), dim=1)
    assert ((w.double() - ref).abs() <= 2e-4 * ref).all()
    ctx.close()
