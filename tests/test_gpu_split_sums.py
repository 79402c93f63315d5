"""Sums over the slabs of a split reduction (router top-k, combine) at every number of slabs, and work lists of very
unequal lengths: layer output against the oracle and, bit for bit, against the staged calls; routing against fp64
logits."""
import ctypes as C

import numpy as np
import pytest

import workloads as wl
from oracle import moe_oracle as orc

import gpu_util as gu

pytestmark = pytest.mark.gpu


class _Plan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("cls", "bm", "bn", "mt_max", "nt1", "nt2", "grid1", "grid2")] + [("w_stream", C.c_bool)]


def _slabs_and_list_workgroups(s):
    """What the host decides for a layer call of this shape: (slabs of the second GEMM, workgroups that build its two
    work lists)."""
    import paper_2605_19945_amd as moe
    lib = moe.load_library()
    make, pick_class, split = lib._Z14gemm_make_planiliii, lib._Z15gemm_pick_classd, lib._Z16gemm_pick_split2RK8GemmPlanliiim
    make.restype, make.argtypes = _Plan, [C.c_int, C.c_int64, C.c_int, C.c_int, C.c_int]
    pick_class.restype, pick_class.argtypes = C.c_int, [C.c_double]
    split.restype, split.argtypes = C.c_int, [C.c_void_p, C.c_int64, C.c_int, C.c_int, C.c_int, C.c_size_t]
    rows = s.T * min(s.k, s.E_local)
    plan = make(pick_class(s.T * s.k / s.E), rows, s.E_local, s.d, s.f)
    part_bytes = min(8 * rows * s.d * 4, 64 << 20)
    blocks = tuple(min(64, -(-g // 256)) for g in (plan.grid1, plan.grid2))
    return split(C.byref(plan), rows, s.E_local, s.d, s.f, part_bytes), blocks


def _layer_and_staged(inp):
    import torch
    import paper_2605_19945_amd as moe
    s = inp.shape
    ctx = moe.MoEContext(max(1, s.T), s.d, s.f, s.E, s.k, s.e_lo, s.E_local, 0)
    x, rp = gu.to_dev_bf16(inp.x), ctx.moe_pack_router(gu.to_dev(inp.Wg))
    packed = ctx.moe_pack_weights(gu.to_dev_bf16(inp.W1), gu.to_dev_bf16(inp.W3), gu.to_dev_bf16(inp.W2))
    out = ctx.moe_layer_forward(x, rp, None, packed)
    layer_idx = ctx.moe_layer_intermediates(s.T)[0].cpu().numpy()
    idx, w, _ = ctx.moe_route(x, rp)
    xp, offsets, row_of, _ = ctx.moe_permute(x, idx)
    y = ctx.moe_grouped_ffn(xp, offsets, ctx.rows_capacity(s.T), packed)
    staged = ctx.moe_combine(y, row_of, w)
    torch.cuda.synchronize()
    ctx.close()
    return out, staged, layer_idx


# f / 64 K steps: 2 to 8 ranges of at least 16 K steps divide them; 16 and 31 cannot be split.  `lists`: workgroups
# that build the work lists of the two GEMMs (256 entries each): one for either list, several for one of them and one
# for the other, both ways round, and the 64 that a list gets at most (its workgroups then build several rounds).
@pytest.mark.parametrize("T,d,f,slabs,lists", [
    (1, 128, 2048, 2, (1, 1)), (3, 128, 3072, 3, (1, 1)), (1, 128, 4096, 4, (1, 1)), (1, 192, 5120, 5, (1, 1)),
    (2, 128, 6144, 6, (2, 1)), (2, 128, 7168, 7, (2, 1)), (5, 128, 8192, 8, (2, 1)), (1, 128, 1024, 1, (1, 1)),
    (1, 128, 1984, 1, (1, 1)), (700, 64, 4096, 1, (2, 1)), (700, 4096, 64, 1, (1, 1)), (1500, 64, 4096, 1, (3, 1)),
    (1500, 8192, 64, 1, (1, 3)), (8000, 64, 32768, 1, (64, 1))])
def test_layer_equals_oracle_and_staged_calls(T, d, f, slabs, lists):
    import torch
    print(f"T={T} d={d} f={f}", flush=True)
    inp = wl.custom("split_sums", T, d, f, 4, 2, seed=T + f, wg_std=0.05, w_std=0.03)
    assert _slabs_and_list_workgroups(inp.shape) == (slabs, lists)
    out, staged, idx = _layer_and_staged(inp)
    assert torch.equal(out.view(torch.int16), staged.view(torch.int16))
    # both build their lists with the same code, so the rows are also compared with the oracle: all of them, or about
    # 400 spread over all row tiles (every column of a row then shows every weight-row tile of both GEMMs)
    tokens = np.unique(np.linspace(0, T - 1, min(T, 400)).astype(np.int64))
    ref = orc.layer_forward(inp.x, inp.Wg, None, inp.W1, inp.W3, inp.W2, 2, tokens=tokens, idx=idx)["out"]
    gu.check_output(gu.f64_of_bf16(out)[tokens], ref, what=f"T={T} d={d} f={f}")


# The reduction over d is cut into the most ranges, up to 8, that divide its K steps of 64 and leave at least 8 of them,
# as these T do not fill the device: 448 and 512 are not split, the others in 2, 3, 4, 5, 6, 7 and 8 slabs
@pytest.mark.parametrize("d", [448, 512, 1024, 1536, 2048, 2560, 3072, 3584, 4096])
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
