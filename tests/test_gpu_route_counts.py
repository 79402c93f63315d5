"""Counts of the routers between the resident and the GEMM path: consecutive calls of one context hand sub-counters and a
ticket from launch to launch, at one workgroup, at fewer and more than there are sub-counters, and with T off the group
size; every call's counts are the histogram of its own indices, and a call that does not ask for counts leaves no trace."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,E,k", [(192, 8, 2), (128, 1, 1), (320, 9, 3), (5120, 16, 1), (448, 17, 4), (64, 31, 16)])
def test_counts_of_consecutive_calls(d, E, k):
    import torch
    import paper_2605_19945_amd as moe
    print(f"d={d} E={E} k={k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(d + E)
    ctx = moe.MoEContext(3001, d, 64, E, k)
    rp = ctx.moe_pack_router(torch.randn(d, E, device="cuda", generator=g))
    packed = ctx.moe_pack_weights(*(torch.randn(*s, device="cuda", generator=g).mul_(0.05).bfloat16()
                                    for s in ((E, d, 64), (E, d, 64), (E, 64, d))))
    x = torch.randn(3001, d, device="cuda", generator=g).bfloat16()
    results = []
    for n, T in enumerate([1, 16, 17, 3001, 511, 512, 513, 2, 3000, 31, 32, 33] * 4):
        if n % 5 == 4:
            ctx.moe_layer_forward(x[:T], rp, None, packed)   # small batches: the router does not count
        idx, _, counts = ctx.moe_route(x[:T], rp)
        results.append((T, idx, counts))
    torch.cuda.synchronize()
    ctx.close()
    for n, (T, idx, counts) in enumerate(results):
        hist = np.bincount(idx.cpu().numpy().ravel(), minlength=E)
        assert counts.cpu().numpy().tolist() == hist.tolist(), f"call {n} (T={T})"
