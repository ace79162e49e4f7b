"""Workloads of the ScMoE forward library, each one a call (or the four operator calls) as a
user's program makes it: what goes in, one pass through the public entry points, what comes
out, what the pass cannot do without, and the same result in 64 bits from plain PyTorch.

A case is a dict of
  form     "scmoe"  one block forward, y = SE(x_cur) + sum_i G(x_prev)_i E_i(x_prev)
           "topk"   the standard top-k MoE layer on x
           "steps"  gate, dispatch, expert FFN and combine as four calls (a program that puts
                    work of its own, for instance an exchange between GPUs, in between)
  T, d, F, E, k     tokens, model width, hidden width, experts, experts per token
  cf                capacity factor; 0: no token is dropped
  dtype             "bf16" or "f32"
  tanh, normalize, biases, cg, residual, zipf, streams, routing   options of the layer; zipf
                    is the exponent of the load over the experts (0: balanced), routing asks
                    for copies of the routing arrays
"""
import math

import torch

from paper_2404_05019_amd import binding as B

DEV = "cuda:0"


def _case(form, T, d, F, E, k=1, cf=1.25, dtype="bf16", tanh=False, normalize=0, biases=False, cg=0, residual=False,
          zipf=0.0, streams=1, routing=False):
    return dict(form=form, T=T, d=d, F=F, E=E, k=k, cf=cf, dtype=dtype, tanh=tanh, normalize=normalize, biases=biases,
                cg=cg, residual=residual, zipf=zipf, streams=streams, routing=routing)


def listed():
    cases = [
        # the smallest configuration, fp32: latency and launches
        ("tiny_f32", _case("scmoe", 256, 64, 256, 4, dtype="f32")),
        # a decode step of a GPT-style layer for a batch of 8: nothing is dropped, weights are streamed
        ("decode_8", _case("scmoe", 8, 2048, 8192, 16, cf=0.0)),
        # a larger decode batch, shared expert on a second stream
        ("decode_64_streams", _case("scmoe", 64, 2048, 8192, 16, cf=0.0, streams=2)),
        # a chunk of a prompt between two decode steps, an odd number of tokens, with biases
        ("chunk_500", _case("scmoe", 500, 2048, 8192, 16, cf=0.0, biases=True)),
        # a vision layer (SwinV2-MoE-S stage 3)
        ("small", _case("scmoe", 8192, 384, 1536, 8)),
        # the same widths in fp32 with biases and a coefficient gate
        ("small_f32", _case("scmoe", 2048, 384, 1536, 8, dtype="f32", biases=True, cg=1)),
        # GPT-style layers: balanced, skewed load with drops, and the large headline configuration
        ("medium", _case("scmoe", 16384, 1024, 4096, 8)),
        ("skewed", _case("scmoe", 16384, 1024, 4096, 16, cf=1.0, zipf=1.2, routing=True)),
        ("large", _case("scmoe", 32768, 2048, 8192, 16)),
        # the standard top-2 layer the shortcut layer is compared with
        ("top2_medium", _case("topk", 16384, 1024, 4096, 8, k=2, normalize=1)),
        # ScMoE-2 with the second coefficient gate and the residual, ragged sizes, tanh GELU
        ("scmoe2_ragged", _case("scmoe", 3001, 768, 3072, 12, k=2, tanh=True, biases=True, cg=2, residual=True)),
        # the operators one by one, many small experts
        ("steps_e32", _case("steps", 4096, 1024, 2048, 32, k=2, normalize=1)),
    ]
    return [dict(c, name=n) for n, c in cases]


def _generic(c):
    """Whether the widths or the type keep the call off the bf16 matrix-core kernels (which take multiples of 64)."""
    return c["dtype"] == "f32" or c["d"] % 64 != 0 or c["F"] % 64 != 0


def draw(rng):
    """One more layer of these ranges: 1 to 32768 tokens, widths 64 to 2048, 2 to 64 experts."""
    while True:
        form = rng.choice(["scmoe", "scmoe", "scmoe", "topk", "steps"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        step = rng.choice([64, 64, 64, 8])
        T = int(round(math.exp(rng.uniform(0.0, math.log(32768)))))
        d = max(64, int(round(math.exp(rng.uniform(math.log(64), math.log(2048))) / step)) * step)
        F = max(step, int(round(d * rng.choice([2, 8 / 3, 4]) / step)) * step)
        E = rng.choice([2, 4, 8, 8, 12, 16, 16, 24, 32, 64])
        k = rng.choice([1, 1, 1, 2, 2, 3, 4])
        if k > E:
            continue
        c = _case(form, T, d, F, E, k, cf=rng.choice([0.0, 1.0, 1.25, 1.25, 2.0]) if T > 64 else 0.0, dtype=dtype,
                  tanh=rng.random() < 0.2, normalize=rng.randrange(2), biases=rng.random() < 0.4,
                  cg=rng.choice([0, 0, 1, 2]) if form == "scmoe" else 0, residual=form == "scmoe" and rng.random() < 0.3,
                  zipf=rng.choice([0.0, 0.0, 0.0, 1.2]) if T >= 256 else 0.0,
                  streams=rng.choice([1, 1, 2]) if form == "scmoe" else 1, routing=form != "steps" and rng.random() < 0.2)
        big = listed()[8]
        w, most = work(c), work(big)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"] * (0.01 if _generic(c) else 0.9):
            return c


# ---- inputs ---------------------------------------------------------------------------------------


def _torch_type(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _inputs(c, seed):
    """Activations ~ N(0, 1) and weights ~ N(0, 0.02) in the layer's type; gate matrix and biases in fp32."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    T, d, F, E, tt = c["T"], c["d"], c["F"], c["E"], _torch_type(c)

    def normal(*shape, scale=0.02, dtype=torch.float32):
        if len(shape) == 3:                       # expert by expert: no fp32 copy of all weights
            out = torch.empty(shape, dtype=dtype, device=DEV)
            for q in range(shape[0]):
                out[q] = torch.randn(shape[1:], generator=g, device=DEV) * scale
            return out
        return (torch.randn(shape, generator=g, device=DEV) * scale).to(dtype)

    shared = c["form"] == "scmoe"
    x = dict(x=normal(T, d, scale=1.0, dtype=tt), Wg=normal(d, E), W1=normal(E, F, d, dtype=tt), W2=normal(E, d, F, dtype=tt))
    x["x_cur"] = normal(T, d, scale=1.0, dtype=tt) if shared else None
    x["W1s"] = normal(F, d, dtype=tt) if shared else None
    x["W2s"] = normal(d, F, dtype=tt) if shared else None
    x["b1"] = normal(E, F) if c["biases"] else None
    x["b2"] = normal(E, d) if c["biases"] else None
    x["b1s"] = normal(F) if c["biases"] and shared else None
    x["b2s"] = normal(d) if c["biases"] and shared else None
    x["Wcg"] = normal(c["cg"], d) if c["cg"] else None
    x["residual"] = normal(T, d, scale=1.0, dtype=tt) if c["residual"] else None
    x["bias"] = None
    if c["zipf"]:
        # an additive gate term under which the experts' loads follow (e + 1) ** -zipf
        z = x["x"].float() @ x["Wg"]
        sigma = z.std()
        q = torch.arange(1, E + 1, device=DEV, dtype=torch.float32) ** -c["zipf"]
        q /= q.sum()
        b = sigma * torch.log(q)
        for _ in range(40):
            load = torch.bincount((z + b).argmax(1), minlength=E).float() / T
            b = b + 0.5 * sigma * torch.log(q / load.clamp_min(1e-4))
        x["bias"] = (b - b.max()).contiguous()
    return x


def _capacity(c):
    """Rows an expert accepts: ceil(cf k T / E), in whole numbers (cf is a multiple of 1 / 100)."""
    if not c["cf"]:
        return c["T"] * c["k"]
    return -(-round(c["cf"] * 100) * c["k"] * c["T"] // (100 * c["E"]))


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    T, d, F, E, k, tt = c["T"], c["d"], c["F"], c["E"], c["k"], _torch_type(c)
    C = _capacity(c)
    code = B.BF16 if c["dtype"] == "bf16" else B.F32
    gelu = B.GELU_TANH if c["tanh"] else B.GELU_ERF
    rows = max(1, min(T * k, E * C))
    s = dict(case=c, x=x, y=torch.zeros(T, d, dtype=tt, device=DEV))
    i32 = lambda n, v=0: torch.full((n,), v, dtype=torch.int32, device=DEV)  # noqa: E731
    if c["form"] == "steps" or c["routing"]:
        s["out"] = dict(expert_idx=i32(T * k), gate_w=torch.zeros(T * k, device=DEV), counts=i32(E), offsets=i32(E + 1),
                        dst_row=i32(T * k))
    if c["form"] == "steps":
        s.update(C=C, gelu=gelu, rows=rows, src_token=i32(rows, -1), probs=torch.zeros(T, E, device=DEV),
                 x_perm=torch.zeros(rows, d, dtype=tt, device=DEV), y_perm=torch.zeros(rows, d, dtype=tt, device=DEV),
                 hidden=torch.empty(rows, B.scmoe_padded_ld(F, code), dtype=tt, device=DEV)[:, :F],
                 ws=torch.empty(max(16, B.scmoe_dispatch_workspace_bytes(T, E, k)), dtype=torch.uint8, device=DEV),
                 ws_ffn=torch.empty(max(16, B.scmoe_expert_ffn_workspace_bytes(code, d, F)), dtype=torch.uint8, device=DEV))
        return s
    s["desc"] = B.make_desc(T, d, F, E, k, C, code, gelu, c["normalize"], c["cg"])
    s["weights"] = B.make_weights(x["Wg"], x["W1"], x["W2"], x["W1s"], x["W2s"], x["bias"], x["b1"], x["b2"], x["b1s"],
                                  x["b2s"], x["Wcg"])
    s["ws"] = torch.empty(B.scmoe_workspace_bytes(s["desc"]), dtype=torch.uint8, device=DEV)
    s["routing"] = B.make_routing_out(**s["out"]) if c["routing"] else None
    s["aux"] = torch.cuda.Stream() if c["streams"] == 2 else None
    return s


def run(state):
    s = state
    c, x = s["case"], s["x"]
    if c["form"] == "scmoe":
        B.scmoe_layer_forward(s["desc"], x["x"], x["x_cur"], s["weights"], s["y"], s["ws"], residual=x["residual"],
                              routing=s["routing"], stream_aux=s["aux"])
    elif c["form"] == "topk":
        B.moe_topk_layer_forward(s["desc"], x["x"], s["weights"], s["y"], s["ws"], routing=s["routing"])
    else:
        o = s["out"]
        B.scmoe_gate_topk(x["x"], x["Wg"], x["bias"], c["k"], o["expert_idx"], o["gate_w"], s["probs"], c["normalize"])
        B.scmoe_dispatch(x["x"], o["expert_idx"], c["E"], c["k"], s["C"], o["counts"], o["offsets"], o["dst_row"],
                         s["src_token"], s["x_perm"], s["ws"])
        B.scmoe_expert_ffn(s["x_perm"], o["offsets"], s["rows"], x["W1"], x["b1"], x["W2"], x["b2"], s["hidden"],
                           s["y_perm"], s["gelu"], s["ws_ffn"])
        B.scmoe_combine(s["y_perm"], o["dst_row"], o["gate_w"], c["k"], None, None, None, s["y"])
        return dict(o, y=s["y"], probs=s["probs"], src_token=s["src_token"], x_perm=s["x_perm"], y_perm=s["y_perm"])
    return dict(s["out"], y=s["y"]) if c["routing"] else s["y"]


# ---- what a pass cannot do without ----------------------------------------------------------------


def _kept(c):
    """Expected packed rows and experts with a row."""
    n, E, C = c["T"] * c["k"], c["E"], _capacity(c)
    q = [(e + 1.0) ** -c["zipf"] for e in range(E)]
    share = [v / sum(q) for v in q]
    return sum(min(n * p, C) for p in share), sum(1.0 - (1.0 - p) ** n for p in share)


def work(case):
    c = case
    T, d, F, E, k = c["T"], c["d"], c["F"], c["E"], c["k"]
    eb = 2 if c["dtype"] == "bf16" else 4
    K, active = _kept(c)
    shared = c["form"] == "scmoe"
    flops = 4.0 * (K + (T if shared else 0)) * d * F + 2.0 * T * d * E
    acts = T * d * (2 + shared + c["residual"])                    # x, x_cur and the residual in, y out
    if c["form"] == "steps":
        acts += 4 * K * d                                          # x_perm and y_perm are results of one call and inputs of the next
    size = (acts + 2 * (active + shared) * d * F) * eb + 4 * d * (E + c["cg"])
    if c["biases"]:
        size += 4 * (active + shared) * (d + F)
    if c["form"] == "steps" or c["routing"]:
        size += 4 * (3 * T * k + 2 * E + 1)
    if c["form"] == "steps":
        size += 4 * (K + T * E)
    return {"bytes": float(size), "flops": float(flops)}


def tolerance(case):
    # Routing is whole numbers and has to be the same.  fp32: sums in another order.  bf16: the
    # hidden rows, the experts' outputs and y are stored in 8 bits of mantissa.
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1}


# ---- the same in 64 bits ----------------------------------------------------------------------------


def _logits(x, Wg, bias):
    """Gate logits as the interface defines them, because they decide whole numbers: a chain of fused
    multiply-adds in fp32 over ascending features (product and sum in 64 bits, rounded to 32 at each step)."""
    xt, w = x.double().t().contiguous(), Wg.double()
    acc = torch.zeros(x.shape[0], Wg.shape[1], dtype=torch.float64, device=x.device)
    for i in range(Wg.shape[0]):
        acc = torch.addcmul(acc, xt[i].unsqueeze(1), w[i].unsqueeze(0)).float().double()
    return acc if bias is None else (acc.float() + bias).double()


def _mlp(x, W1, b1, W2, b2, tanh):
    """W2 . GELU(W1 . x + b1) + b2 in 64 bits, at most 4096 rows at a time."""
    w1, w2 = W1.double(), W2.double()
    parts = []
    for p in x.double().split(4096):
        h = p @ w1.t()
        if b1 is not None:
            h = h + b1.double()
        h = torch.nn.functional.gelu(h, approximate="tanh" if tanh else "none") @ w2.t()
        parts.append(h if b2 is None else h + b2.double())
    return torch.cat(parts)


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    T, E, k, C = c["T"], c["E"], c["k"], _capacity(c)
    logits = _logits(x["x"], x["Wg"], x["bias"])
    idx = torch.sort(logits, dim=1, descending=True, stable=True)[1][:, :k]
    probs = torch.softmax(logits, 1)
    w = torch.softmax(logits.gather(1, idx), 1) if c["normalize"] else probs.gather(1, idx)
    # items in the order of choices, then tokens; the first C of an expert are kept
    items = idx.t().reshape(-1)
    tokens = torch.arange(T, device=DEV).repeat(k)
    factor = w.t().reshape(-1)
    y = torch.zeros(T, c["d"], dtype=torch.float64, device=DEV)
    x_perm, y_perm = [], []
    for e in range(E):
        at = (items == e).nonzero().flatten()[:C]
        if at.numel() == 0:
            continue
        rows = x["x"][tokens[at]]
        out = _mlp(rows, x["W1"][e], None if x["b1"] is None else x["b1"][e], x["W2"][e], None if x["b2"] is None else x["b2"][e], c["tanh"])
        y.index_add_(0, tokens[at], out * factor[at].unsqueeze(1))
        if c["form"] == "steps":
            x_perm.append(rows.double())
            y_perm.append(out)
    if c["form"] == "scmoe":
        s = _mlp(x["x_cur"], x["W1s"], x["b1s"], x["W2s"], x["b2s"], c["tanh"])
        if c["cg"]:
            g = x["x_cur"].double() @ x["Wcg"].double().t()
            if c["cg"] == 1:
                s = s * torch.sigmoid(g)
            else:
                g = torch.softmax(g, 1)
                s, y = s * g[:, :1], y * g[:, 1:]
        y = y + s
    if x["residual"] is not None:
        y = y + x["residual"].double()
    if c["form"] != "steps":
        return dict(y=y, gate_w=w.reshape(-1), expert_idx=None, counts=None, offsets=None, dst_row=None) if c["routing"] else y
    left = max(1, min(T * k, E * C)) - sum(p.shape[0] for p in x_perm)
    pad = torch.zeros(left, c["d"], dtype=torch.float64, device=DEV)
    return dict(y=y, gate_w=w.reshape(-1), probs=probs, x_perm=torch.cat(x_perm + [pad]), y_perm=torch.cat(y_perm + [pad]),
                expert_idx=None, counts=None, offsets=None, dst_row=None, src_token=None)
