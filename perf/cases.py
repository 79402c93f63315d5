"""The work this library does for its users, as cases that can be timed and compared.

A case is one call path through the public entry points (`MoEContext` methods of `paper_2605_19945_amd`) on one
shape, one token load and one kind of expert load:

* mode "layer":  `moe_layer_forward`, the whole per-GPU MoE layer -- what a serving step calls;
* mode "staged": `moe_route`, `moe_permute`, `moe_grouped_ffn`, `moe_combine` one after the other, as a program
  that puts its own exchange between dispatch and experts calls them;
* mode "ffn":    `moe_grouped_ffn` alone on rows that another GPU has already routed (expert parallelism);
* mode "route":  consecutive `moe_route` calls whose counts become the rows of an expert-utilisation trace.

Shapes are those of `workloads/gen.py`, `bench.py` and the tests: "mixtral" (8 experts, top-2), "fine" (128 small
experts, top-8), "mid" (64 experts, top-8), "wide" (16 wide experts, top-1), "ep" (one GPU's 32 of 256 experts,
top-8), "tiny" (the smoke-test layer); drawn cases add free shapes of the same ranges.  Inputs are synthetic:
Gaussian activations and weights of the scales the tests use, router biases that give the expert loads described
in `workloads/gen.py`.
"""
import math

import torch

import paper_2605_19945_amd as moe

# d, f, E, k, standard deviation of the router matrix (None: 1/sqrt(d), unit-variance logits), kind of router bias
SHAPES = {
    "tiny": dict(d=128, f=256, E=8, k=2, wg=0.02, load="even"),
    "mixtral": dict(d=4096, f=14336, E=8, k=2, wg=0.02, load="even"),
    "fine": dict(d=2048, f=768, E=128, k=8, wg=None, load="biased"),
    "mid": dict(d=4096, f=3072, E=64, k=8, wg=None, load="biased"),
    "wide": dict(d=5120, f=8192, E=16, k=1, wg=None, load="biased"),
    "ep": dict(d=7168, f=2048, E=256, k=8, wg=None, load="share"),
    "trace": dict(d=512, f=64, E=8, k=2, wg=None, load="consistent"),
}
EP_LO, EP_LOCAL = 64, 32  # resident experts of the expert-parallel share
W_STD = 0.02              # standard deviation of the expert weights
T_SERVE = 4096            # token capacity a serving context is created with (more if the case needs more)
MAX_FLOPS = 6.0 * 8192 * 8 * 4096 * 3072  # of the largest listed case
MAX_T = 16384             # the largest per-GPU token load that is profiled


def _case(name, mode, shape, T, **more):
    c = dict(mode=mode, shape=shape, T=T, steps=1, E_local=0, e_lo=0)
    c.update(SHAPES[shape])
    c["wg"] = c["wg"] or 1.0 / math.sqrt(c["d"])
    if shape == "ep":
        c.update(e_lo=EP_LO, E_local=EP_LOCAL)
    c.update(more)
    c["E_local"] = c["E_local"] or c["E"]
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest layer there is (smoke test, unit tests, toy models): launches and host work only
        _case("tiny_T64", "layer", "tiny", 64),
        # one user's decode step: two experts' weights are streamed for one token
        _case("mixtral_T1", "layer", "mixtral", 1),
        # a decode batch: every expert's weights once
        _case("mixtral_T64", "layer", "mixtral", 64),
        # a small prefill under the skew described for real traffic (consistent and temporal experts), ragged
        _case("mixtral_skewed_T1000", "layer", "mixtral", 1000, load="skewed"),
        # an ordinary prefill chunk, near-even load: the benchmark's default workload
        _case("mixtral_T4096", "layer", "mixtral", 4096),
        # a decode batch of a model with many small experts: about five rows per expert, odd size
        _case("fine_T77", "layer", "fine", 77),
        # prefill of the same model
        _case("fine_T8192", "layer", "fine", 8192),
        # one GPU's share of an expert-parallel layer, medium batch: the router sees 256 experts, 32 live here
        _case("ep_T2048", "layer", "ep", 2048),
        # the largest: prefill over 64 medium experts, top-8
        _case("mid_T8192", "layer", "mid", 8192),
        # the four stages called one by one (a program that exchanges rows between GPUs in between), odd size,
        # few wide experts, top-1
        _case("staged_wide_T3001", "staged", "wide", 3001),
        # the receiving side of expert parallelism: already-routed rows, Zipf-distributed over the local experts
        _case("ffn_ep_N5003", "ffn", "ep", 5003),
        # a 16-step expert-utilisation trace of a small router: counts of consecutive calls in one matrix
        _case("trace_16x256", "route", "trace", 256, steps=16),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _flops_per_token(c):
    local = c["T"] * c["k"] if c["load"] != "share" else 0.75 * c["T"]  # (see _local_share)
    if c["mode"] == "ffn":
        local = c["T"]
    return 6.0 * local * c["d"] * c["f"] / c["T"] + 2.0 * c["d"] * c["E"]


def draw(rng):
    kind = rng.choice(["mixtral", "mixtral", "skewed", "fine", "mid", "wide", "ep", "free", "free", "ffn", "route"])
    mode = "staged" if rng.random() < 0.25 else "layer"
    if kind == "free":
        # any shape the library takes, up to the widths of the named ones
        E = rng.choice([4, 6, 8, 12, 16, 24, 32, 48, 60, 64, 96])
        k = min(E, rng.choice([1, 2, 2, 4, 6, 8]))
        c = _case("", mode, "tiny", 1, d=64 * _log_uniform(rng, 2, 80), f=64 * _log_uniform(rng, 2, 128), E=E, k=k,
                  E_local=E, load=rng.choice(["even", "biased"]))
        c["shape"], c["wg"] = "free", 1.0 / math.sqrt(c["d"])
        while 3.0 * E * c["d"] * c["f"] > 1.5e9:  # the expert weights of the largest named shape
            c["f"] = max(64, c["f"] // 2 // 64 * 64)
    elif kind == "ffn":
        c = _case("", "ffn", "ep", 1)
    elif kind == "route":
        c = _case("", "route", "trace", 1, d=64 * _log_uniform(rng, 4, 112), E=rng.choice([8, 8, 16]), steps=rng.randint(4, 24))
        c["E_local"], c["wg"] = c["E"], 1.0 / math.sqrt(c["d"])
    elif kind == "skewed":
        c = _case("", mode, "mixtral", 1, load="skewed")
    else:
        c = _case("", mode, kind, 1)
    most = MAX_T if c["mode"] != "route" else 2048
    if c["mode"] == "ffn":
        most = 4 * MAX_T
    most = max(1, min(most, int(MAX_FLOPS / _flops_per_token(c))))
    c["T"] = _log_uniform(rng, 1, most)
    return c


# ---- inputs -------------------------------------------------------------------------------------------
def _bias(c, seed):
    """Router bias of every expert (None: none), as a CPU tensor: it sets the expected load of each expert."""
    E, load = c["E"], c["load"]
    if load == "even":
        return None
    if load == "biased":
        return torch.randn(E, generator=torch.Generator().manual_seed(7919 * seed + 3)) * 0.5
    b = torch.zeros(E)
    if load == "share":  # Zipf popularity over the resident experts
        for r in range(c["E_local"]):
            b[c["e_lo"] + r] = 1.5 - math.log(r + 1)
    elif load == "skewed":  # experts 0, 1 lead always; the others follow a Zipf law
        b[0] = b[1] = 2.4
        for e in range(2, E):
            b[e] = -1.2 * math.log(e - 1)
    else:  # "consistent": two experts of a small router lead in every step
        b[1] = b[6] = 1.5
    return b


def _zipf_offsets(N, E_local, seed):
    """Offsets of N rows split over the local experts with Zipf(1) probabilities, drawn from the seed."""
    p = 1.0 / torch.arange(1, E_local + 1, dtype=torch.float64)
    pick = torch.multinomial(p, N, replacement=True, generator=torch.Generator().manual_seed(seed))
    off = torch.zeros(E_local + 1, dtype=torch.int32)
    off[1:] = torch.cumsum(torch.bincount(pick, minlength=E_local), 0)
    return off


def _untie(x, Wg, bias, k):
    """A token whose k-th and next logit lie within 3e-5 of each other may go to either expert, depending on the order
    of fp32 sums (two of 8192 tokens over 64 experts did, against fp64 logits).  Such tokens, at most a few in ten
    thousand, get the values of one without a tie, so that two correct passes can be compared row by row."""
    if k >= Wg.shape[1]:
        return
    logits = x.double() @ Wg.double()
    if bias is not None:
        logits += bias
    top = logits.topk(k + 1, dim=1).values
    tied = top[:, k - 1] - top[:, k] < 3e-5
    x.copy_(torch.where(tied[:, None], x[torch.argmin(tied.to(torch.int32))], x))


def _inputs(c, seed):
    """The raw inputs of a case, made from the seed alone: the rows of "ffn", or router matrix, bias and activations,
    and the expert weights W1, W3, W2 (none for "route")."""
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(1000003 * seed + 17)
    T, d, f, E, k, El = c["T"], c["d"], c["f"], c["E"], c["k"], c["E_local"]

    def normal(*shape, dtype=torch.bfloat16, std=1.0):
        return torch.empty(shape, dtype=dtype, device=dev).normal_(0.0, std, generator=g)

    r = {}
    if c["mode"] == "ffn":
        # rows arrive expert-contiguous; the host knows how many it received
        r["xp"], r["offsets"] = normal(T, d), _zipf_offsets(T, El, seed).to(dev)
    else:
        Wg = normal(d, E, dtype=torch.float32, std=c["wg"])
        bias = _bias(c, seed)
        xs = [normal(T, d) for _ in range(c["steps"])]
        if c["load"] == "skewed":  # two pairs of temporal experts, each busy for one stretch of the tokens
            for pair, lo, hi in (((2, 3), 0.20, 0.35), ((4, 5), 0.60, 0.75)):
                u = normal(d, dtype=torch.float32)
                u /= u.norm()
                t0, t1 = round(lo * T), round(hi * T)
                for x in xs:
                    x[t0:t1] = (x[t0:t1].float() + 20.0 * u).to(torch.bfloat16)
                for e in pair:
                    Wg[:, e] += 0.5 * u
        r["bias"] = None if bias is None else bias.to(dev)
        for x in xs:
            _untie(x, Wg, r["bias"], k)
        r["xs"], r["Wg"] = xs, Wg
    if c["mode"] != "route":
        r["experts"] = [normal(El, d, f, std=W_STD), normal(El, d, f, std=W_STD), normal(El, f, d, std=W_STD)]
    return r


def prepare(case, seed):
    c = dict(case)
    T, d, f, E, k, El = c["T"], c["d"], c["f"], c["E"], c["k"], c["E_local"]
    r = _inputs(c, seed)
    s = dict(mode=c["mode"], T=T)
    if c["mode"] == "ffn":
        ctx = moe.MoEContext(max(1, -(-T // k)), d, f, E, k, c["e_lo"], El)
        s["xp"], s["offsets"] = r["xp"], r["offsets"]
    else:
        t_max = T if c["shape"] in ("tiny", "free", "trace") else max(T, T_SERVE)
        ctx = moe.MoEContext(t_max, d, f, E, k, c["e_lo"], El)
        s["bias"], s["xs"], s["router"] = r["bias"], r["xs"], ctx.moe_pack_router(r["Wg"])
        s["counts"] = torch.zeros(c["steps"], E, dtype=torch.int32, device="cuda")
    if c["mode"] != "route":
        s["packed"] = ctx.moe_pack_weights(*r["experts"])
    s["ctx"] = ctx
    return s


def run(s):
    ctx = s["ctx"]
    if s["mode"] == "layer":
        return ctx.moe_layer_forward(s["xs"][0], s["router"], s["bias"], s["packed"], counts_out=s["counts"][0])
    if s["mode"] == "ffn":
        return ctx.moe_grouped_ffn(s["xp"], s["offsets"], s["T"], s["packed"])
    if s["mode"] == "route":
        got = [ctx.moe_route(x, s["router"], s["bias"], counts=s["counts"][i]) for i, x in enumerate(s["xs"])]
        return [t for idx, w, _ in got for t in (idx, w)] + [s["counts"]]
    x = s["xs"][0]
    idx, w, _ = ctx.moe_route(x, s["router"], s["bias"], counts=s["counts"][0])
    xp, offsets, row_of, _ = ctx.moe_permute(x, idx)
    y = ctx.moe_grouped_ffn(xp, offsets, ctx.rows_capacity(s["T"]), s["packed"])
    return ctx.moe_combine(y, row_of, w)


# ---- the same results in 64 bits ---------------------------------------------------------------------------
def _ffn64(r, rows, e):
    """Rows of one expert through its SwiGLU network, in 64 bits."""
    W1, W3, W2 = (w[e].double() for w in r["experts"])
    g = rows @ W1
    return (g * torch.sigmoid(g) * (rows @ W3)) @ W2


def exact(case, seed):
    c = dict(case)
    r = _inputs(c, seed)
    if c["mode"] == "ffn":
        off, y = r["offsets"].tolist(), torch.zeros(c["T"], c["d"], dtype=torch.float64, device="cuda")
        for e in range(c["E_local"]):
            if off[e + 1] > off[e]:
                y[off[e]:off[e + 1]] = _ffn64(r, r["xp"][off[e]:off[e + 1]].double(), e)
        return y
    routed = []
    for x in r["xs"]:
        logits = x.double() @ r["Wg"].double()
        if r["bias"] is not None:
            logits += r["bias"].double()
        top = logits.topk(c["k"], dim=1)
        routed.append((top.indices, torch.softmax(top.values, dim=1)))
    if c["mode"] == "route":
        counts = torch.stack([torch.bincount(i.reshape(-1), minlength=c["E"]) for i, _ in routed])
        return [t for i, w in routed for t in (i.to(torch.int32), w)] + [counts.to(torch.int32)]
    x, (idx, w) = r["xs"][0], routed[0]
    out = torch.zeros(c["T"], c["d"], dtype=torch.float64, device="cuda")
    for e in range(c["E_local"]):
        tok, slot = (idx == c["e_lo"] + e).nonzero(as_tuple=True)
        if tok.numel():
            out.index_add_(0, tok, w[tok, slot, None] * _ffn64(r, x[tok].double(), e))
    return out


# ---- what a pass cannot do without, and how closely two correct passes agree --------------------------------
_expected = {}


def _local_share(c):
    """(assignments per token to resident experts, probability of each resident expert to be picked by a token), from
    4096 sampled logit rows: Gaussian logits plus the bias."""
    key = (c["load"], c["E"], c["k"], c["e_lo"], c["E_local"], c["d"])
    if key not in _expected:
        logits = torch.randn(4096, c["E"], generator=torch.Generator().manual_seed(1)) * c["wg"] * math.sqrt(c["d"])
        bias = _bias(c, 0)
        if bias is not None:
            logits += bias
        picks = torch.bincount(logits.topk(c["k"], dim=1).indices.reshape(-1), minlength=c["E"]) / 4096.0
        local = picks[c["e_lo"]:c["e_lo"] + c["E_local"]]
        _expected[key] = (float(local.sum()), local.tolist())
    return _expected[key]


def work(case):
    c = case
    T, d, f, E, k = c["T"], c["d"], c["f"], c["E"], c["k"]
    if c["mode"] == "route":
        per_step = 2.0 * T * d + 8.0 * T * k + 4.0 * E + 4.0 * d * E
        return {"bytes": per_step * c["steps"], "flops": 2.0 * T * d * E * c["steps"]}
    if c["mode"] == "ffn":
        rows, touched, router = float(T), sum(1.0 for n in _zipf_offsets(T, c["E_local"], 0).diff().tolist() if n), 0.0
        moved = 4.0 * rows * d
    else:
        per_token, p = _local_share(c)
        rows = per_token * T
        touched = sum(1.0 - (1.0 - min(1.0, q)) ** T for q in p)
        router, moved = 2.0 * T * d * E, 4.0 * T * d + 4.0 * d * E
    return {"bytes": moved + 6.0 * d * f * touched, "flops": 6.0 * rows * d * f + router}


def tolerance(case):
    if case["mode"] == "route":
        # gate weights: fp32 sums of bf16 activations times a router matrix kept to 2^-18; the slots of two selected
        # experts change places where their logits tie to the last bits
        return {"rel": 2e-5, "max": 1e-3, "differ": 1e-3}
    # The intermediate, the expert rows and the output are rounded to bf16 once each.  Measured over the listed cases:
    # against fp64 without those roundings 2.9e-3 (largest element 0.034), with the same roundings and other
    # sums 5e-4 (0.023).
    return {"rel": 1e-2, "max": 0.1}
