"""Performance cases of the MoE block: the calls a training or serving program
makes through the package's public entry points, over the sizes it makes them
at.

A case is a dict of plain values: `kind` names the entry points (train:
MoEBlock.forward + backward; infer: MoEInfer.forward; lora: MoELoRA.forward +
backward; experts: MoEExperts.forward + backward), the rest are sizes and
options.  Inputs are drawn on the GPU from the seed alone: x, dY ~ N(0, 1),
weights ~ N(0, 0.02^2), rounded to bf16, as the repository's own workloads
draw them.
"""
import math

import torch

import paper_2608_00916_amd as moe

_QWEN = dict(H=2048, E=128, k=8, F=768)  # the expert layer of a 30B-A3B MoE model
_TRAIN = dict(mask=False, zipf=0.0, dw_fp32=False, recompute=False, aux=0.0, z=0.0)


def listed():
    return [
        # One training step of a toy layer: nothing but launches and latency.
        dict(name="train_tiny", kind="train", T=256, H=128, E=8, k=2, F=256, **_TRAIN),
        # Serving: one short query-passage pair scored alone.
        dict(name="infer_64", kind="infer", T=64, mask=False, zipf=0.0, **_QWEN),
        # Serving: one passage of the usual maximum length.
        dict(name="infer_512", kind="infer", T=512, mask=False, zipf=0.0, **_QWEN),
        # Serving: a full prefill batch (16 passages of 512 tokens).
        dict(name="infer_8192", kind="infer", T=8192, mask=False, zipf=0.0, **_QWEN),
        # Full fine-tuning, two query groups of 8 passages x 512 tokens: the
        # ordinary training step.
        dict(name="train_8192", kind="train", T=8192, **_QWEN, **_TRAIN),
        # Full fine-tuning with a skewed router: hot experts at 10x the mean,
        # a few without any row.
        dict(name="train_zipf_32768", kind="train", T=32768, **_QWEN, **{**_TRAIN, "zipf": 1.2}),
        # Long passages padded to 4096 tokens, padding masked out of the routing.
        dict(name="train_long_65536", kind="train", T=65536, **_QWEN, **{**_TRAIN, "mask": True}),
        # Adapter fine-tuning of the experts at the usual rank.
        dict(name="lora_8192", kind="lora", T=8192, rank=16, mask=False, **_QWEN),
        # One expert-parallel rank of eight: 16 local experts and the rows
        # dispatched to them.
        dict(name="experts_8359", kind="experts", rows=8359, H=2048, E=16, F=768, dw_fp32=False, recompute=False),
        # A small ragged step with every option of mixed-precision training:
        # odd token count, masked tokens, fp32 weight gradients, recomputed
        # activations, router losses; widths that are no multiple of 256.
        dict(name="train_ragged_3001", kind="train", T=3001, H=640, E=64, k=6, F=384, mask=True, zipf=0.0,
             dw_fp32=True, recompute=True, aux=1e-2, z=1e-3),
        # A layer of twice the widths with fewer experts.
        dict(name="train_wide_4096", kind="train", T=4096, H=4096, E=32, k=4, F=1536, **_TRAIN),
    ]


def draw(rng):
    """One more case: any kind, tokens, widths, experts and options over the
    listed cases' ranges, no costlier than the largest of them."""
    most = max(work(c)["flops"] for c in listed())

    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["train", "train", "infer", "lora", "experts"])
        H = 128 * logint(1, 32)
        F = 128 * logint(2, 12)
        E = 8 * logint(1, 32)
        if rng.random() < 0.4:
            H, F, E = 2048, 768, 128
        k = rng.randint(1, min(E, 10))
        if E * H * F > 128 * 4096 * 1536:
            continue
        c = dict(kind=kind, H=H, E=E, F=F)
        if kind == "experts":
            c.update(rows=logint(64, 65536), dw_fp32=rng.random() < 0.3, recompute=rng.random() < 0.3)
        elif kind == "infer":
            c.update(T=logint(16, 65536), k=k, mask=rng.random() < 0.3, zipf=rng.choice([0.0, 0.0, 1.2]))
        elif kind == "lora":
            c.update(T=logint(256, 32768), k=k, rank=rng.choice([16, 16, 32, 48, 64]), mask=rng.random() < 0.3)
        else:
            loss = rng.random() < 0.25
            c.update(T=logint(256, 65536), k=k, mask=rng.random() < 0.4, zipf=rng.choice([0.0, 0.0, 1.2]),
                     dw_fp32=rng.random() < 0.3, recompute=rng.random() < 0.3, aux=1e-2 if loss else 0.0,
                     z=1e-3 if loss else 0.0)
        if work(c)["flops"] <= most:
            return c


# ------------------------------------------------------------------ inputs
def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape, std=1.0):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)

    H, E, F = case["H"], case["E"], case["F"]
    t = dict(w_gate=normal(E, H, F, std=0.02), w_up=normal(E, H, F, std=0.02), w_down=normal(E, F, H, std=0.02))
    if case["kind"] == "experts":
        rows = case["rows"]
        # counts of a near-uniform router: every row picks one of the E experts
        owner = torch.randint(0, E, (rows,), device="cuda", generator=g)
        t["counts"] = torch.bincount(owner, minlength=E).to(torch.int32)
        t["x"] = normal(rows, H)
        t["dy"] = normal(rows, H)
        return t
    T = case["T"]
    t["x"] = normal(T, H)
    t["w_r"] = normal(H, E, std=0.02)
    t["dy"] = normal(T, H)
    if case.get("zipf"):
        # popularity rank^-s over a random order of the experts, through a
        # constant last channel and its router row; a few experts unused
        rank = torch.empty(E, dtype=torch.float64, device="cuda")
        rank[torch.randperm(E, device="cuda", generator=g)] = torch.arange(1, E + 1, dtype=torch.float64, device="cuda")
        bias = -0.4 * case["zipf"] * rank.log()
        bias[rank > max(case["k"], E - E // 32)] = -1e4
        t["x"][:, H - 1] = 1.0
        t["w_r"][H - 1] = bias.to(torch.bfloat16)
    t["mask"] = None
    if case["mask"]:
        # sequences of a sixteenth of the tokens, each at least half full
        L = max(1, T // 16)
        n = -(-T // L)
        lens = torch.randint((L + 1) // 2, L + 1, (n,), device="cuda", generator=g)
        pos = torch.arange(L, device="cuda")
        t["mask"] = (pos[None, :] < lens[:, None]).reshape(-1)[:T].to(torch.uint8).contiguous()
    if case["kind"] == "lora":
        r = case["rank"]
        for n, s in dict(a1=(E, H, r), b1_gate=(E, r, F), b1_up=(E, r, F), a2=(E, F, r), b2=(E, r, H)).items():
            t[n] = normal(*s, std=0.05)
    return t


_ADAPTERS = ("a1", "b1_gate", "b1_up", "a2", "b2")
_SCALE = 2.0  # alpha / r of the adapters


def prepare(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "experts":
        blk = moe.MoEExperts(case["rows"], case["H"], case["E"], case["F"], case["dw_fp32"], case["recompute"])
        return dict(kind=kind, blk=blk, t=t)
    size = (case["T"], case["H"], case["E"], case["F"], case["k"])
    st = dict(kind=kind, t=t)
    if kind == "infer":
        st["blk"] = moe.MoEInfer(*size, mask=case["mask"])
    elif kind == "lora":
        st["blk"] = moe.MoELoRA(*size, case["rank"], mask=case["mask"])
        st["lora"] = moe.lora_args(case["rank"], _SCALE, *(t[n] for n in _ADAPTERS))
    else:
        st["blk"] = moe.MoEBlock(*size, mask=case["mask"], dw_fp32=case["dw_fp32"], recompute=case["recompute"],
                                 aux_loss_coef=case["aux"], z_loss_coef=case["z"])
        st["loss"] = bool(case["aux"] or case["z"])
    return st


def run(state):
    blk, t, kind = state["blk"], state["t"], state["kind"]
    if kind == "experts":
        o = blk.forward(t["x"], t["counts"], t["w_gate"], t["w_up"], t["w_down"])
        return (o, *blk.backward(t["x"], t["w_gate"], t["w_up"], t["w_down"], t["dy"]))
    w = (t["w_r"], t["w_gate"], t["w_up"], t["w_down"])
    if kind == "infer":
        return blk.forward(t["x"], *w, t["mask"])
    if kind == "lora":
        y = blk.forward(t["x"], *w, state["lora"], t["mask"])
        return (y, *blk.backward(t["x"], *w, state["lora"], t["dy"]))
    y = blk.forward(t["x"], *w, t["mask"])
    out = (y, *blk.backward(t["x"], *w, t["dy"]))
    return (*out, blk.views["router_loss"]) if state["loss"] else out


# ------------------------------------------------------------------ work, tolerance
def work(case):
    """Operations of the expert and router products over the routed rows;
    bytes of every input and output once.  A masked case routes three
    quarters of its tokens (the mean of its sequence lengths)."""
    H, E, F, kind = case["H"], case["E"], case["F"], case["kind"]
    if kind == "experts":
        R = case["rows"]
        weights = 3 * E * H * F
        grads = weights * (4 if case["dw_fp32"] else 2)
        # + A and, kept, G and U for the backward
        return dict(bytes=2 * (4 * R * H + 2 * weights) + grads, flops=18 * H * F * R)
    T = case["T"]
    Tv = 0.75 * T if case["mask"] else T
    R = Tv * case["k"]
    # an expert without a row needs no weights: at most R of them are read
    weights = 3 * min(E, R) * H * F + H * E
    if kind == "infer":
        return dict(bytes=2 * (2 * T * H + weights), flops=6 * H * F * R + 2 * H * E * Tv)
    if kind == "lora":
        r = case["rank"]
        adapters = E * r * (2 * H + 3 * F)
        # forward and data gradients of the base, the adapters in both and
        # their own gradients; the router forward and its part of dX
        flops = 12 * H * F * R + 6 * r * (2 * H + 3 * F) * R + 4 * H * E * Tv
        return dict(bytes=2 * (4 * T * H + 2 * weights) + 2 * 2 * adapters + 2 * adapters, flops=flops)
    grads = (3 * E * H * F + H * E) * (4 if case["dw_fp32"] else 2)
    return dict(bytes=2 * (4 * T * H + 2 * weights) + grads, flops=18 * H * F * R + 6 * H * E * Tv)


def tolerance(case):
    """bf16 activations, gradients and outputs; fp32 sums.  Every output was
    0.0035 to 0.0046 from the 64-bit values at the listed and drawn cases: four
    times that."""
    return {"rel": 1.6e-2}


# ------------------------------------------------------------------ the same in 64 bits
def exact(case, seed):
    t = {n: (v if v is None or not v.is_floating_point() else v.double()) for n, v in _inputs(case, seed).items()}
    kind, E = case["kind"], case["E"]
    x, dy = t["x"], t["dy"]
    if kind == "experts":
        ends = t["counts"].cumsum(0).tolist()
        starts = [0] + ends[:-1]
        o, dx = torch.zeros_like(x), torch.zeros_like(x)
        dwg, dwu, dwd = (torch.zeros_like(t[n]) for n in ("w_gate", "w_up", "w_down"))
        for e in range(E):
            s = slice(starts[e], ends[e])
            if starts[e] == ends[e]:
                continue
            f = _expert_fwd(x[s], t["w_gate"][e], t["w_up"][e], t["w_down"][e])
            o[s] = f["o"]
            dx[s], dwg[e], dwu[e], dwd[e] = _expert_bwd(x[s], f, t["w_gate"][e], t["w_up"][e], t["w_down"][e], dy[s])
        return (o, dx, dwg, dwu, dwd)

    T, k = case["T"], case["k"]
    z = x @ t["w_r"]
    on = torch.ones(T, dtype=torch.bool, device=x.device) if t["mask"] is None else t["mask"] != 0
    # selection on the fp32 logits, ties to the lower expert
    idx = z.float().sort(dim=1, descending=True, stable=True).indices[:, :k]
    gates = torch.softmax(z.gather(1, idx), dim=1)
    y, dx = torch.zeros_like(x), torch.zeros_like(x)
    dg = torch.zeros_like(gates)
    train = kind != "infer"
    lora = kind == "lora"
    names = _ADAPTERS if lora else ("w_gate", "w_up", "w_down")
    dw = {n: torch.zeros_like(t[n]) for n in names} if train else {}
    for e in range(E):
        tok, slot = torch.nonzero((idx == e) & on[:, None], as_tuple=True)
        if tok.numel() == 0:
            continue
        xe = x[tok]
        we = [t[n][e] for n in ("w_gate", "w_up", "w_down")]
        if lora:
            a1, b1g, b1u, a2, b2 = (t[n][e] for n in _ADAPTERS)
            we = [we[0] + _SCALE * a1 @ b1g, we[1] + _SCALE * a1 @ b1u, we[2] + _SCALE * a2 @ b2]
        f = _expert_fwd(xe, *we)
        g = gates[tok, slot][:, None]
        y.index_add_(0, tok, g * f["o"])
        if not train:
            continue
        dg[tok, slot] = (dy[tok] * f["o"]).sum(1)
        dxe, dwg, dwu, dwd = _expert_bwd(xe, f, *we, g * dy[tok])
        dx.index_add_(0, tok, dxe)
        if lora:  # W = base + scale a b:  da = scale dW b^T, db = scale a^T dW
            dw["a1"][e] = _SCALE * (dwg @ b1g.T + dwu @ b1u.T)
            dw["b1_gate"][e] = _SCALE * a1.T @ dwg
            dw["b1_up"][e] = _SCALE * a1.T @ dwu
            dw["a2"][e] = _SCALE * dwd @ b2.T
            dw["b2"][e] = _SCALE * a2.T @ dwd
        else:
            dw["w_gate"][e], dw["w_up"][e], dw["w_down"][e] = dwg, dwu, dwd
    if not train:
        return y
    dzs = gates * (dg - (gates * dg).sum(1, keepdim=True)) * on[:, None]
    dz = torch.zeros_like(z).scatter_(1, idx, dzs)
    loss = None
    if case.get("aux") or case.get("z"):
        tv = on.sum().double()
        f = torch.bincount(idx[on].reshape(-1), minlength=E).double() / (tv * k)
        p = torch.softmax(z, 1) * on[:, None]
        lse = torch.logsumexp(z, 1) * on
        loss = torch.stack([case["aux"] * E * (f * p.sum(0) / tv).sum(), case["z"] * (lse ** 2).sum() / tv])
        dz = dz + case["aux"] * E / tv * p * (f - p @ f[:, None]) + case["z"] * 2 / tv * lse[:, None] * p
    dx += dz @ t["w_r"].T
    if lora:
        return (y, dx, *(dw[n] for n in _ADAPTERS))
    out = (y, dx, x.T @ dz, dw["w_gate"], dw["w_up"], dw["w_down"])
    return out if loss is None else (*out, loss)


def _expert_fwd(x, wg, wu, wd):
    g, u = x @ wg, x @ wu
    s = torch.sigmoid(g)
    a = g * s * u
    return dict(g=g, u=u, s=s, a=a, o=a @ wd)


def _expert_bwd(x, f, wg, wu, wd, d_o):
    g, u, s = f["g"], f["u"], f["s"]
    da = d_o @ wd.T
    dg = da * u * s * (1.0 + g * (1.0 - s))
    du = da * g * s
    return dg @ wg.T + du @ wu.T, x.T @ dg, x.T @ du, f["a"].T @ d_o
