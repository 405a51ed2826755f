"""What is timed when the framework's speed is looked at: the calls that its users make.

A case is a dict of plain values: `kind` says which calls, the rest are sizes and options.

  stack   a schedule of mixing layers: forward and backward (or the forward alone)
  layer   one mixing layer, forward and backward
  lm      one training step of the byte language model (embedding, stack, head, all gradients)
  attn    one attention layer of the hybrid schedules (projections and core), both directions
  shared  the channel-shared stack, both directions
  field   one application of the field coupling, both directions
  decode  one window, position after position, through the stack

listed() holds the shapes of the repository's own workloads and tests, and small and ragged
ones beside them; draw() spreads the same calls over the sizes between.
"""
import math

import torch

from paper_2609_18145_amd import hcmix

DT = {"bf16": torch.bfloat16, "f32": torch.float32}
VOCAB = 256
HEAD_DIM = 64


def listed():
    return [
        # the smallest calls: the tiny fp32 workload through autograd, where launches count
        dict(name="tiny_f32", kind="stack", dtype="f32", n=16, width=32, batch=2, layers=4,
             sched="rot", causal=False, train=True, autograd=True),
        # one layer at a ragged shape: a few short windows, a width of no large tile
        dict(name="layer_w192", kind="layer", dtype="bf16", n=64, width=192, batch=5, layer=3,
             causal=True),
        # the reach task (width 64, the whole stack in one launch per direction)
        dict(name="reach", kind="stack", dtype="bf16", n=256, width=64, batch=64, layers=8,
             sched="rot", causal=False, train=True, autograd=False),
        # fp32 training, an ordinary size: full precision for those who compare against it
        dict(name="stack_f32", kind="stack", dtype="f32", n=256, width=256, batch=16, layers=8,
             sched="rot", causal=True, train=True, autograd=False),
        # a bf16 width that is a multiple of 8 and not of 64
        dict(name="stack_w200", kind="stack", dtype="bf16", n=256, width=200, batch=32, layers=8,
             sched="rot", causal=True, train=True, autograd=False),
        # a few prompts through the sparse layers of the window-256 hybrid (8 local, 6 jumps)
        dict(name="prefill_b3", kind="stack", dtype="bf16", n=256, width=512, batch=3, layers=14,
             sched="hybrid", causal=True, train=False, autograd=False),
        # the language model's training step at the window-256 workload's full size
        dict(name="lm_step", kind="lm", n=256, width=512, batch=64, layers=16),
        # the long window: strides up to 2048 rows, activations in HBM
        dict(name="long4096", kind="stack", dtype="bf16", n=4096, width=1024, batch=8, layers=24,
             sched="rot", causal=True, train=True, autograd=False),
        # an attention layer of the hybrids, 8 heads of 64
        dict(name="attn_layer", kind="attn", n=256, width=512, heads=8, batch=64),
        # the channel-shared stack of the window-256 workload (bound by memory)
        dict(name="shared256", kind="shared", dtype="bf16", n=256, width=512, batch=64, layers=16,
             sched="rot", causal=True),
        # one application of the field coupling at the window-256 workload's size
        dict(name="field256", kind="field", n=256, width=512, coords=32, batch=64, scaled=True),
        # generation: every position of 64 windows, one at a time
        dict(name="decode256", kind="decode", dtype="bf16", n=256, width=512, batch=64,
             layers=16, sched="rot"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["stack", "stack", "stack", "layer", "lm", "attn", "shared", "field",
                       "decode"])
    if kind in ("stack", "layer"):
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        n = 1 << rng.randint(4, 12 if dtype == "bf16" else 9)
        if dtype == "f32":
            width = _log(rng, 16, 384)
        elif rng.random() < 0.3:
            width = 8 * _log(rng, 5, 40)   # narrower ones round too coarsely for deep stacks
        else:
            width = 64 * _log(rng, 1, 16)
        layers = 1 if kind == "layer" else rng.randint(2, 24 if width >= 64 else 12)
        # at most the long window's work, an eighth of it off the matrix-core widths
        most = 8 * 4096 * 1024 ** 2 * 24 // (1 if dtype == "bf16" and width % 64 == 0 else 64)
        batch = _log(rng, 1, max(1, min(512, 65536 // n, most // (n * width ** 2 * layers))))
        causal = rng.random() < 0.7
        if kind == "layer":
            return dict(kind=kind, dtype=dtype, n=n, width=width, batch=batch,
                        layer=rng.randint(0, 15), causal=causal)
        sched = rng.choice(["rot", "rot", "hybrid"]) if causal else "rot"
        return dict(kind=kind, dtype=dtype, n=n, width=width, batch=batch, layers=layers,
                    sched=sched, causal=causal, train=rng.random() < 0.7,
                    autograd=rng.random() < 0.3)
    if kind == "lm":
        return dict(kind=kind, n=1 << rng.randint(5, 8), width=128 * rng.randint(1, 4),
                    batch=_log(rng, 1, 64), layers=rng.randint(2, 16))
    if kind == "attn":
        heads = rng.randint(1, 8)
        return dict(kind=kind, n=32 * rng.randint(1, 8), width=HEAD_DIM * heads, heads=heads,
                    batch=_log(rng, 1, 64))
    if kind == "shared":
        dtype = rng.choice(["bf16", "f32"])
        return dict(kind=kind, dtype=dtype, n=1 << rng.randint(4, 8),
                    width=64 * rng.randint(1, 8), batch=_log(rng, 1, 64),
                    layers=rng.randint(2, 16), sched="rot", causal=rng.random() < 0.7)
    if kind == "field":
        return dict(kind=kind, n=rng.randint(16, 256), width=64 * rng.randint(1, 8),
                    coords=rng.randint(2, 64), batch=_log(rng, 1, 64),
                    scaled=rng.random() < 0.7)
    return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]), n=1 << rng.randint(4, 8),
                width=64 * rng.randint(1, 8), batch=_log(rng, 1, 64), layers=rng.randint(2, 16),
                sched=rng.choice(["rot", "hybrid"]))


# ---- inputs ----

def _schedule(c):
    """Layer codes: the rotated schedule, or the window-256 hybrid's alternation of local layers
    and jumps, longest first."""
    L, n = c["layers"], c["n"]
    if c["sched"] == "rot":
        return list(range(L))
    b = n.bit_length() - 1
    return [hcmix.LAYER_NEAR if l % 2 == 0 else (b - 1 - (l // 2) % b) for l in range(L)]


def _inputs(c, seed):
    """The call's operands, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape, std=1.0, dtype=torch.float32):
        return (torch.randn(*shape, generator=g, device="cuda") * std).to(dtype)

    k = c["kind"]
    n, w, B = c["n"], c["width"], c["batch"]
    if k in ("stack", "layer", "decode"):
        dt = DT[c["dtype"]]
        L = c.get("layers", 1)
        return dict(x=normal(B, n, w, dtype=dt), dy=normal(B, n, w, dtype=dt),
                    ws=normal(L, w, w, std=w ** -0.5, dtype=dt),
                    wo=normal(L, w, w, std=w ** -0.5, dtype=dt))
    if k == "lm":
        L, bf = c["layers"], torch.bfloat16
        p = torch.arange(1, VOCAB + 1, device="cuda", dtype=torch.float32) ** -1.1
        p = p[torch.randperm(VOCAB, generator=g, device="cuda")]
        seq = torch.multinomial(p, B * (n + 1), replacement=True, generator=g)
        seq = seq.view(B, n + 1).to(torch.int32)
        # weights of half the usual variance: the two maps' sum then keeps the activations'
        # scale, and the softmax is that of a model in training and not one saturated row
        return dict(tokens=seq[:, :n].contiguous(), targets=seq[:, 1:].contiguous(),
                    table=normal(VOCAB, w, dtype=bf), head=normal(VOCAB, w, std=w ** -0.5, dtype=bf),
                    bias=normal(VOCAB, std=0.1),
                    ws=normal(L, w, w, std=(2 * w) ** -0.5, dtype=bf),
                    wo=normal(L, w, w, std=(2 * w) ** -0.5, dtype=bf))
    if k == "attn":
        bf, hw = torch.bfloat16, c["heads"] * HEAD_DIM
        return dict(x=normal(B, n, w, dtype=bf), dy=normal(B, n, w, dtype=bf),
                    wqkv=normal(3 * hw, w, std=w ** -0.5, dtype=bf),
                    wout=normal(w, hw, std=hw ** -0.5, dtype=bf))
    if k == "shared":
        dt = DT[c["dtype"]]
        return dict(x=normal(B, n, w, dtype=dt), dy=normal(B, n, w, dtype=dt),
                    tables=normal(c["layers"], n, n, std=0.5 ** 0.5))
    # field: a mean squared distance of 100 between positions
    bf = torch.bfloat16
    return dict(x=normal(B, n, w, dtype=bf), dy=normal(B, n, w, dtype=bf),
                p=normal(B, n, c["coords"], std=(50.0 / c["coords"]) ** 0.5))


def prepare(case, seed):
    """Inputs, weights, and the buffers that a training or serving loop keeps."""
    c = case
    s = dict(_inputs(c, seed), case=c)
    k = c["kind"]
    n, w, B = c["n"], c["width"], c["batch"]
    dev = torch.device("cuda", torch.cuda.current_device())

    def f32(*shape):
        return torch.empty(*shape, dtype=torch.float32, device=dev)

    if k in ("stack", "lm", "decode"):
        L = c["layers"]
        s["codes"] = _schedule(c) if k != "lm" else list(range(L))
        s["w_selfs"], s["w_offs"] = list(s["ws"].unbind(0)), list(s["wo"].unbind(0))
    if k == "stack":
        dt = DT[c["dtype"]]
        if c["autograd"] and c["train"]:
            s["leaves"] = [t.clone().requires_grad_(True)
                           for t in (s["x"], *s["w_selfs"], *s["w_offs"])]
            return s
        s["acts"] = torch.empty(L, B, n, w, dtype=dt, device=dev)
        s["outs"] = list(s["acts"].unbind(0))
        if c["train"]:
            s["dw"] = f32(2, L, w, w)
            s["dws"], s["dwo"] = (list(t.unbind(0)) for t in s["dw"].unbind(0))
            s["dx"] = torch.empty_like(s["x"])
            s["work"] = hcmix.alloc_stack_workspace(B, n, w, L, dt, dev)
    elif k == "layer":
        dt = DT[c["dtype"]]
        s["w_self"], s["w_off"] = s["ws"][0], s["wo"][0]
        s["y"], s["dx"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
        s["dw_self"], s["dw_off"] = f32(w, w), f32(w, w)
        s["work"] = hcmix.alloc_workspace(B, n, w, dt, dev)
    elif k == "lm":
        bf = torch.bfloat16
        s["x0"] = torch.empty(B, n, w, dtype=bf, device=dev)
        s["outs"] = list(torch.empty(L, B, n, w, dtype=bf, device=dev).unbind(0))
        s["dw"] = f32(2, L, w, w)
        s["dws"], s["dwo"] = (list(t.unbind(0)) for t in s["dw"].unbind(0))
        s["dx"] = torch.empty_like(s["x0"])
        s["work"] = hcmix.alloc_stack_workspace(B, n, w, L, bf, dev)
        s["targets"] = s["targets"].view(-1)
    elif k == "shared":
        L = c["layers"]
        s["codes"] = _schedule(c)
        s["tabs"] = list(s["tables"].unbind(0))
        s["acts"] = torch.empty(L, B, n, w, dtype=DT[c["dtype"]], device=dev)
        s["outs"] = list(s["acts"].unbind(0))
        s["dt"] = f32(L, n, n)
        s["dts"] = list(s["dt"].unbind(0))
        s["dx"] = torch.empty_like(s["x"])
    elif k == "field":
        s["work"] = torch.empty(hcmix.field_workspace_bytes(B, n, c["coords"]),
                                dtype=torch.uint8, device=dev)
        s["y"], s["dx"], s["dp"] = (torch.empty_like(s[t]) for t in ("x", "x", "p"))
    elif k == "decode":
        s["cols"] = [s["x"][:, i].contiguous() for i in range(n)]
        s["cache"] = hcmix.alloc_decode_cache(B, n, w, s["codes"], DT[c["dtype"]], dev)
        s["ys"] = torch.empty(n, B, w, dtype=DT[c["dtype"]], device=dev)
        s["outs"] = list(s["ys"].unbind(0))
    return s


# ---- one pass ----

def run(state):
    s = state
    c = s["case"]
    k = c["kind"]
    if k == "stack":
        if c["autograd"] and c["train"]:
            y = hcmix.Stack.apply(s["leaves"][0], s["codes"], c["causal"], *s["leaves"][1:])
            grads = torch.autograd.grad(y, s["leaves"], s["dy"])
            L = c["layers"]
            return dict(y=y, dx=grads[0], dw=torch.stack(grads[1:]).view(2, L, *grads[1].shape))
        xs = hcmix.stack_forward(s["x"], s["w_selfs"], s["w_offs"], s["codes"], c["causal"],
                                 outs=s["outs"])
        if not c["train"]:
            return dict(acts=s["acts"])
        hcmix.stack_backward(xs, s["w_selfs"], s["w_offs"], s["codes"], s["dy"], c["causal"],
                             dx=s["dx"], dws=s["dws"], dwo=s["dwo"], workspace=s["work"])
        return dict(acts=s["acts"], dx=s["dx"], dw=s["dw"])
    if k == "layer":
        y = hcmix.forward(s["x"], s["w_self"], s["w_off"], c["layer"], c["causal"], out=s["y"])
        dx, dws, dwo = hcmix.backward(s["x"], s["w_self"], s["w_off"], s["dy"], c["layer"],
                                      c["causal"], dx=s["dx"], dw_self=s["dw_self"],
                                      dw_off=s["dw_off"], workspace=s["work"])
        return dict(y=y, dx=dx, dws=dws, dwo=dwo)
    if k == "lm":
        w, rows = c["width"], c["batch"] * c["n"]
        x0 = hcmix.embedding_forward(s["table"], s["tokens"], out=s["x0"])
        xs = hcmix.stack_forward(x0, s["w_selfs"], s["w_offs"], s["codes"], True, outs=s["outs"])
        top = xs[-1].view(rows, w)
        loss, dlog, dbias = hcmix.head_cross_entropy(top, s["head"], s["bias"], s["targets"],
                                                     1.0 / rows, with_dbias=True)
        gx, dhead = hcmix.head_backward(top, s["head"], dlog)
        hcmix.stack_backward(xs, s["w_selfs"], s["w_offs"], s["codes"],
                             gx.view(c["batch"], c["n"], w), True, dx=s["dx"], dws=s["dws"],
                             dwo=s["dwo"], workspace=s["work"])
        dtable = hcmix.embedding_backward(s["tokens"], s["dx"], VOCAB)
        return dict(loss=loss, dlogits=dlog, dbias=dbias, dhead=dhead, dtable=dtable, dw=s["dw"])
    if k == "attn":
        B, n, w, h = c["batch"], c["n"], c["width"], c["heads"]
        x, dy = s["x"].view(B * n, w), s["dy"].view(B * n, w)
        qkv = hcmix.linear_forward(x, s["wqkv"]).view(B, n, 3, h, HEAD_DIM)
        o, lse = hcmix.attention_forward(qkv)
        y = hcmix.linear_forward(o.view(B * n, -1), s["wout"])
        do, dwout = hcmix.linear_backward(o.view(B * n, -1), s["wout"], dy)
        dqkv = hcmix.attention_backward(qkv, o, lse, do.view(B, n, h, HEAD_DIM))
        dx, dwqkv = hcmix.linear_backward(x, s["wqkv"], dqkv.view(B * n, -1))
        return dict(y=y, dx=dx, dwqkv=dwqkv, dwout=dwout)
    if k == "shared":
        xs = hcmix.shared_stack_forward(s["x"], s["tabs"], s["codes"], c["causal"],
                                        outs=s["outs"])
        hcmix.shared_stack_backward(xs, s["tabs"], s["codes"], s["dy"], c["causal"], dx=s["dx"],
                                    dtables=s["dts"])
        return dict(acts=s["acts"], dx=s["dx"], dt=s["dt"])
    if k == "field":
        y, m, lse, _ = hcmix.field_forward(s["p"], s["x"], 1.0, c["scaled"], y=s["y"],
                                           workspace=s["work"])
        dp, dx = hcmix.field_backward(s["p"], s["x"], m, lse, s["dy"], 1.0, c["scaled"],
                                      dp=s["dp"], dx=s["dx"], workspace=s["work"],
                                      reuse_table=True)
        return dict(y=y, row_mean=m, lse=lse, dp=dp, dx=dx)
    for pos in range(c["n"]):
        hcmix.decode_step(s["cols"][pos], s["w_selfs"], s["w_offs"], s["codes"], c["n"], pos,
                          s["cache"], out=s["outs"][pos])
    return dict(ys=s["ys"])


# ---- what a pass cannot do without ----

def work(case):
    c = case
    k = c["kind"]
    n, w, B = c["n"], c["width"], c["batch"]
    rows = B * n

    def links(code, causal):   # products with a weight matrix per position
        if code == hcmix.LAYER_NEAR:
            return 2 - 1 / n
        return 1.5 if causal else 2

    if k in ("stack", "layer", "decode"):
        es = 2 if c["dtype"] == "bf16" else 4
        codes = [c["layer"]] if k == "layer" else _schedule(c)
        L = len(codes)
        fl = sum(2 * rows * w * w * links(q, c.get("causal", True)) for q in codes)
        if k == "decode":   # every step reads every weight it uses: no less without keeping them
            return dict(bytes=2 * rows * w * es + 2 * L * w * w * es, flops=fl)
        train = k == "layer" or c["train"]
        kept = L if k == "layer" or not (c["autograd"] and train) else 1
        by = (1 + kept) * rows * w * es + 2 * L * w * w * es
        if train:
            out_es = es if k == "stack" and c["autograd"] else 4
            by += 2 * rows * w * es + 2 * L * w * w * out_es
        return dict(bytes=by, flops=3 * fl if train else fl)
    if k == "lm":
        L = c["layers"]
        fl = 3 * L * 3 * rows * w * w + 3 * 2 * rows * w * VOCAB
        by = (rows * (4 + 4 + 4 + 2 * VOCAB) + VOCAB * (w * (2 + 2 + 4 + 4) + 8)
              + 2 * L * w * w * (2 + 4))
        return dict(bytes=by, flops=fl)
    if k == "attn":
        hw = c["heads"] * HEAD_DIM
        core = B * c["heads"] * n * (n + 1) / 2 * HEAD_DIM * 2
        return dict(bytes=4 * rows * w * 2 + 4 * hw * w * (2 + 4),
                    flops=3 * 2 * rows * w * 4 * hw + core * (2 + 5))
    if k == "shared":
        es, L = (2 if c["dtype"] == "bf16" else 4), c["layers"]
        return dict(bytes=(L + 3) * rows * w * es + L * n * n * 4 + 2 * L * n * 4,
                    flops=L * rows * w * 2 * 2 * (3 if c["causal"] else 4) / 2 * 1.5)
    pairs = B * n * (n + 1) / 2
    return dict(bytes=4 * rows * w * 2 + 2 * rows * c["coords"] * 4 + 2 * rows * 4,
                flops=pairs * 2 * (3 * w + 4 * c["coords"]))


def tolerance(case):
    """About four times the error against 64 bits that each kind of call was measured to have.
    In 16 bits every layer rounds its output once, so a stack's grows with the root of its
    depth: 0.0017 for one layer, 0.0047 for 8, 0.0066 for 16, 0.0082 for 24."""
    c = case
    if c.get("dtype") == "f32":
        return {"rel": 1e-5}                 # sums of 32 bits: 1.4e-6 after 8 layers
    if c["kind"] in ("stack", "layer", "decode"):
        return {"rel": 0.005 + 0.005 * math.sqrt(c.get("layers", 1))}
    # lm 0.0028, attn 0.0043, shared 0.0027, field 0.0023
    return {"rel": {"lm": 0.012, "attn": 0.018, "shared": 0.011, "field": 0.01}[c["kind"]]}


# ---- the same in 64 bits, in plain torch ----

def _partner(x, code):
    """(partner's vector of every position, 1 where the causal form keeps it)"""
    B, n, w = x.shape
    i = torch.arange(n, device=x.device)
    if code == hcmix.LAYER_NEAR:
        p = torch.cat([torch.zeros_like(x[:, :1]), x[:, :-1]], 1)
        return p, (i >= 1).to(x.dtype)
    d = code % (n.bit_length() - 1)
    return x[:, i ^ (1 << d)], ((i >> d) & 1).to(x.dtype)


def _mix(x, ws, wo, code, causal):
    p, m = _partner(x, code)
    return x @ ws.T + ((p * m[:, None]) if causal else p) @ wo.T


def exact(case, seed):
    c = case
    k = c["kind"]
    raw = _inputs(c, seed)
    f = {q: t.double() for q, t in raw.items() if t.is_floating_point()}
    n, w, B = c["n"], c["width"], c["batch"]

    if k in ("stack", "layer", "decode"):
        codes = [c["layer"]] if k == "layer" else _schedule(c)
        train = k == "layer" or (k == "stack" and c["train"])
        x, ws, wo = (f[q].requires_grad_(train) for q in ("x", "ws", "wo"))
        h, acts = x, []
        for l, code in enumerate(codes):
            h = _mix(h, ws[l], wo[l], code, c.get("causal", True))
            acts.append(h.detach())
        if k == "decode":
            return dict(ys=h.transpose(0, 1).contiguous())
        if not train:
            return dict(acts=torch.stack(acts))
        dx, dws, dwo = torch.autograd.grad(h, (x, ws, wo), f["dy"])
        if k == "layer":
            return dict(y=acts[-1], dx=dx, dws=dws[0], dwo=dwo[0])
        dw = torch.stack([dws, dwo])
        if c["autograd"]:
            return dict(y=acts[-1], dx=dx, dw=dw)
        return dict(acts=torch.stack(acts), dx=dx, dw=dw)
    if k == "lm":
        table, ws, wo, head, bias = (f[q].requires_grad_(True)
                                     for q in ("table", "ws", "wo", "head", "bias"))
        h = table[raw["tokens"].long()]
        for l in range(c["layers"]):
            h = _mix(h, ws[l], wo[l], l, True)
        logits = h.reshape(B * n, w) @ head.T + bias
        loss = torch.nn.functional.cross_entropy(logits, raw["targets"].reshape(-1).long(),
                                                 reduction="none")
        dlog, dtable, dws, dwo, dhead, dbias = torch.autograd.grad(
            loss.mean(), (logits, table, ws, wo, head, bias))
        return dict(loss=loss.detach(), dlogits=dlog, dbias=dbias, dhead=dhead, dtable=dtable,
                    dw=torch.stack([dws, dwo]))
    if k == "attn":
        h = c["heads"]
        x, wqkv, wout = (f[q].requires_grad_(True) for q in ("x", "wqkv", "wout"))
        q, kk, v = (x @ wqkv.T).view(B, n, 3, h, HEAD_DIM).permute(2, 0, 3, 1, 4).unbind(0)
        sc = q @ kk.transpose(-1, -2).contiguous() / math.sqrt(HEAD_DIM)
        sc = sc.masked_fill(torch.ones(n, n, device=x.device).triu(1).bool(), -math.inf)
        o = (sc.softmax(-1) @ v).transpose(1, 2).reshape(B, n, h * HEAD_DIM)
        y = o @ wout.T
        dx, dwqkv, dwout = torch.autograd.grad(y, (x, wqkv, wout), f["dy"])
        return dict(y=y.detach().view(B * n, w), dx=dx.view(B * n, w), dwqkv=dwqkv, dwout=dwout)
    if k == "shared":
        x, tabs = f["x"].requires_grad_(True), f["tables"].requires_grad_(True)
        h, acts = x, []
        i = torch.arange(n, device=x.device)
        for l, code in enumerate(_schedule(c)):
            d = code % (n.bit_length() - 1)
            p, m = _partner(h, code)
            off = tabs[l][i, i ^ (1 << d)] * (m if c["causal"] else 1.0)
            h = tabs[l][i, i][:, None] * h + off[:, None] * p
            acts.append(h.detach())
        dx, dt = torch.autograd.grad(h, (x, tabs), f["dy"])
        return dict(acts=torch.stack(acts), dx=dx, dt=dt)
    p, x = f["p"].requires_grad_(True), f["x"].requires_grad_(True)
    mask = torch.ones(n, n, device=x.device, dtype=x.dtype).tril()
    D = (p[:, :, None] - p[:, None]).square().sum(-1) * mask
    m = D.sum(-1) / torch.arange(1, n + 1, device=x.device)
    # position 0 sees itself alone: its mean is 0 and all its logits are
    a = -D / torch.where(m == 0, 1.0, m)[..., None] if c["scaled"] else -D
    a = a.masked_fill(mask == 0, -math.inf)
    lse = torch.logsumexp(a, -1)
    y = a.softmax(-1) @ x
    dp, dx = torch.autograd.grad(y, (p, x), f["dy"])
    return dict(y=y.detach(), row_mean=m.detach(), lse=lse.detach(), dp=dp, dx=dx)
