"""The work that SubZero+ fine-tuning has this library do, as cases that can be timed and checked.

Each case is one call (or the two calls that always go together) through the package's public
entry points, on inputs of the shapes the configurations use: the Tiny regression layer, the
OPT-1.3B, LLaMA-7B, OPT-13B and Qwen-32B (LoRA) stacks, plus generic sizes between them.

    listed()            the cases, with a name each
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs on the GPU and the handle a program keeps from step to step
    run(state)          one pass; returns its outputs
    work(case)          bytes and operations of one pass that no implementation can do without
    tolerance(case)     how far two correct implementations may differ
    exact(case, seed)   the same outputs from plain torch in float64
"""
import math

import torch

import paper_2608_15665_amd as zo

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
EPS = 1e-3
BETA1, BETA2, EPS_ADAM, STEP = 0.9, 0.95, 1e-8, 10


def listed():
    return [
        # The Tiny regression layer, one query step's forward and losses: the smallest call, in
        # fp32, all 2q blocks on one input.  Launch latency.
        dict(name="tiny_forward_f32", kind="linear", dtype="f32", T=64, m=256, n=512, r=4, q=4,
             est="central", shared=True, loss=True),
        # An attention projection of OPT-1.3B: an ordinary call of the full-tuning step.
        dict(name="linear_opt1.3b_bf16", kind="linear", dtype="bf16", T=4096, m=2048, n=2048, r=16, q=4,
             est="central", shared=False, loss=False),
        # An attention projection of OPT-13B: the call that the headline step repeats most.
        dict(name="linear_opt13b_bf16", kind="linear", dtype="bf16", T=8192, m=5120, n=5120, r=64, q=8,
             est="central", shared=False, loss=False),
        # The same matrix in the first layer, where every block reads one input.
        dict(name="linear_first_layer_bf16", kind="linear", dtype="bf16", T=8192, m=5120, n=5120, r=64, q=8,
             est="central", shared=True, loss=False),
        # fp16 (the paper's precision) at ragged sizes: a batch that fills no tile, a matrix whose
        # sides are multiples of 8 and no more, with the forward-difference blocks.
        dict(name="linear_ragged_f16", kind="linear", dtype="f16", T=1003, m=3080, n=2056, r=24, q=8,
             est="forward", shared=False, loss=False),
        # fp32 weights and activations at a small model's size.
        dict(name="linear_f32", kind="linear", dtype="f32", T=512, m=2048, n=2048, r=16, q=4,
             est="central", shared=False, loss=False),
        # The adapted v projection of Qwen-32B (grouped heads) under the LoRA scheme.
        dict(name="lora_qwen_v_bf16", kind="lora", dtype="bf16", T=4096, m=1024, n=5120, rl=8, r=4, q=4,
             est="central", shared=False),
        # Attention of one OPT-13B layer for the 16 query blocks.
        dict(name="attention_opt13b_bf16", kind="attention", dtype="bf16", nblk=16, T=8192, seq=512,
             heads=40, kv_heads=40, dh=128),
        # Subspace refresh of one OPT-13B layer's twelve panels.
        dict(name="refresh_opt13b_r64", kind="refresh", d=5120, ffn=20480, r=64),
        # The same at the paper's full-tuning rank, on an OPT-1.3B layer.
        dict(name="refresh_opt1.3b_r128", kind="refresh", d=2048, ffn=8192, r=128),
        # The Adam update of one OPT-13B layer's six matrices.
        dict(name="update_opt13b_bf16", kind="update", dtype="bf16", d=5120, ffn=20480, r=64, q=8),
        # A whole LLaMA-7B layer's forward for the 8 query blocks: what a step repeats per layer.
        dict(name="layer_llama7b_bf16", kind="layer", dtype="bf16", T=4096, seq=256, d=4096, heads=32,
             ffn=11008, r=32, q=4),
    ]


# --------------------------------------------------------------------------- drawn cases
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, dtype, lo, hi):
    """A matrix side: a multiple of 128 (as model sides are) half of the time, else odd sizes
    (16-bit types need multiples of 8)."""
    v = _log_int(rng, lo, hi)
    if rng.random() < 0.5:
        return max(128, v // 128 * 128)
    return max(8, v // 8 * 8) if dtype != "f32" else v


def _blocks(q, est):
    return 2 * q if est == "central" else q + 1


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "lora", "attention", "refresh", "update", "layer"])
    if kind in ("linear", "lora"):
        dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
        top = 4096 if dtype == "f32" else 20480
        c = dict(kind=kind, dtype=dtype, T=_log_int(rng, 64, 8192), m=_side(rng, dtype, 256, top),
                 n=_side(rng, dtype, 256, top), q=rng.randint(1, 8), est=rng.choice(["central", "central", "forward"]),
                 shared=rng.random() < 0.25)
        if kind == "lora":
            c.update(rl=rng.choice([4, 8, 16]), r=rng.choice([2, 4, 4, 8]))
        else:
            c.update(r=min(rng.choice([4, 16, 24, 32, 64, 64, 128]), c["m"], c["n"]), loss=rng.random() < 0.25)
        cap = 1.5e11 if dtype == "f32" else 6e12
        while 2.0 * _blocks(c["q"], c["est"]) * c["T"] * c["m"] * c["n"] > cap:
            c["T"] = c["T"] // 2 + 1
            c["q"] = max(1, c["q"] - 1)
        return c
    if kind == "attention":
        seq, dh = _log_int(rng, 48, 2048), rng.choice([64, 128])
        group = rng.choice([1, 1, 4, 5])
        heads = group * rng.randint(1, 8) * (4 if group == 1 else 1)
        nblk = rng.randint(2, 16)
        per = max(1, min(8192 // seq, int(4e11 / (2.0 * nblk * heads * dh * seq * seq))))
        return dict(kind=kind, dtype=rng.choice(["bf16", "f16"]), nblk=nblk, T=seq * per, seq=seq, heads=heads,
                    kv_heads=heads // group, dh=dh)
    if kind == "refresh":
        d = _log_int(rng, 256, 5120)
        return dict(kind=kind, d=d, ffn=rng.choice([1, 2, 3, 4]) * d + rng.choice([0, 0, 7]),
                    r=rng.choice([4, 16, 24, 32, 64, 96, 128]))
    if kind == "update":
        dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
        d = _side(rng, dtype, 256, 5120 if dtype != "f32" else 3072)
        ffn = _side(rng, dtype, d, 4 * d)
        return dict(kind=kind, dtype=dtype, d=d, ffn=ffn, r=rng.choice([4, 16, 24, 32, 64, 128]), q=rng.randint(1, 8))
    heads, dh = rng.choice([4, 8, 12, 16, 20]), rng.choice([64, 128])
    seq = _log_int(rng, 32, 512)
    d = heads * dh
    return dict(kind="layer", dtype=rng.choice(["bf16", "f16"]), T=seq * max(1, 2048 // seq), seq=seq, d=d,
                heads=heads, ffn=max(64, _log_int(rng, 2 * d, 4 * d) // 32 * 32), r=rng.choice([8, 16, 32]),
                q=rng.randint(1, 4))


# --------------------------------------------------------------------------- inputs
class _Gen:
    """Tensors drawn on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, *shape, dtype=torch.float32, std=1.0):
        t = torch.randn(*shape, generator=self.g, device="cuda", dtype=dtype)
        return t if std == 1.0 else t.mul_(std)

    def orth(self, rows, r):
        """Column-orthonormal rows x r, fp32 (a Gaussian panel divided by its Cholesky factor)."""
        o = self.normal(rows, r).double()
        R = torch.linalg.cholesky(o.t() @ o)
        return torch.linalg.solve_triangular(R, o.t(), upper=False).t().contiguous().float()

    def matrix(self, m, n, r, q, dt):
        return dict(W=self.normal(m, n, dtype=dt, std=0.02), U=self.orth(m, r), V=self.orth(n, r),
                    Z=self.normal(q, r, r))


def _table(q, est):
    """(query, sign) of every block."""
    if est == "central":
        return [b // 2 for b in range(2 * q)], [1 - 2 * (b % 2) for b in range(2 * q)]
    return [0] + list(range(q)), [0] + [1] * q


LAYER = ("q", "k", "v", "o", "gate", "up", "down")


def _layer_sides(c):
    d, f = c["d"], c["ffn"]
    return {"q": (d, d), "k": (d, d), "v": (d, d), "o": (d, d), "gate": (f, d), "up": (f, d), "down": (d, f)}


def _opt_sides(c):
    """The six matrices of an OPT layer."""
    d, f = c["d"], c["ffn"]
    return [(d, d)] * 4 + [(f, d), (d, f)]


def _inputs(c, seed):
    g = _Gen(seed)
    kind = c["kind"]
    dt = DTYPES.get(c.get("dtype"))
    if kind in ("linear", "lora"):
        T, m, n, q = c["T"], c["m"], c["n"], c["q"]
        nx = 1 if c["shared"] else _blocks(q, c["est"])
        s = dict(X=g.normal(nx * T, n, dtype=dt))
        if kind == "linear":
            s.update(g.matrix(m, n, c["r"], q, dt))
            if c["loss"]:
                s["Ystar"] = g.normal(T, m, dtype=dt, std=0.02 * math.sqrt(n))
        else:
            rl, r = c["rl"], min(c["r"], c["rl"])
            s.update(W=g.normal(m, n, dtype=dt, std=0.02), A=g.normal(rl, n, std=0.02), UA=g.orth(rl, r),
                     VA=g.orth(n, r), ZA=g.normal(q, r, r), B=g.normal(m, rl, std=0.02), UB=g.orth(m, r),
                     VB=g.orth(rl, r), ZB=g.normal(q, r, r))
        return s
    if kind == "attention":
        rows, dh = c["nblk"] * c["T"], c["dh"]
        return dict(Q=g.normal(rows, c["heads"] * dh, dtype=dt), K=g.normal(rows, c["kv_heads"] * dh, dtype=dt),
                    V=g.normal(rows, c["kv_heads"] * dh, dtype=dt))
    if kind == "refresh":
        return dict(omega=[g.normal(rows, c["r"]) for mn in _opt_sides(c) for rows in mn])
    if kind == "update":
        items = []
        for m, n in _opt_sides(c):
            it = g.matrix(m, n, c["r"], c["q"], dt)
            it.update(M1=g.normal(c["r"], c["r"], std=0.1), M2=g.normal(c["r"], c["r"], std=0.3).square_())
            items.append(it)
        return dict(items=items, g=g.normal(c["q"]))
    mats = {nm: g.matrix(m, n, c["r"], c["q"], dt) for nm, (m, n) in _layer_sides(c).items()}
    norms = {nm: 1.0 + g.normal(c["d"], std=0.1) for nm in ("rms1_gamma", "rms2_gamma")}
    return dict(mats=mats, norms=norms, H=g.normal(2 * c["q"] * c["T"], c["d"], dtype=dt))


LORA_KEYS = ("A", "UA", "VA", "ZA", "B", "UB", "VB", "ZB")
LR = 1e-3
SCALE = 2.0


def prepare(case, seed):
    c = dict(case)
    s = _inputs(c, seed)
    kind = c["kind"]
    s["case"] = c
    if kind in ("linear", "lora"):
        bq, bs = _table(c["q"], c["est"])
        xs = 0 if c["shared"] else c["T"] * c["n"]
        if kind == "linear":
            s["op"] = zo.PerturbedLinear(s["X"], s["W"], s["U"], s["V"], s["Z"], bq, bs, EPS, c["T"],
                                         x_block_stride=xs)
        else:
            s["op"] = zo.LoraPerturbedLinear(s["X"], s["W"], *[s[k] for k in LORA_KEYS], bq, bs, EPS, SCALE, c["T"],
                                             x_block_stride=xs)
    elif kind == "attention":
        s["out"] = torch.empty_like(s["Q"])
    elif kind == "refresh":
        s["out"] = [torch.empty_like(o) for o in s["omega"]]
    elif kind == "layer":
        bq, bs = _table(c["q"], "central")
        s["op"] = zo.LlamaLayer(s["mats"], s["norms"], bq, bs, EPS, c["T"], c["seq"], c["heads"])
        s["out"] = torch.empty_like(s["H"])
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "linear":
        Y = s["op"]()
        if c["loss"]:
            return Y, zo.sq_loss(Y, s["Ystar"], _blocks(c["q"], c["est"]), c["T"])
        return Y
    if kind == "lora":
        return s["op"]()
    if kind == "attention":
        return zo.causal_attention(s["Q"], s["K"], s["V"], c["nblk"], c["T"], c["seq"], c["heads"], out=s["out"],
                                   kv_heads=c["kv_heads"])
    if kind == "refresh":
        return zo.subspace_refresh(s["omega"], c["r"], out=s["out"])
    if kind == "update":
        zo.subspace_adam_update(s["items"], s["g"], STEP, LR, BETA1, BETA2, EPS_ADAM)
        return [[it["W"], it["M1"], it["M2"]] for it in s["items"]]
    return s["op"](s["H"], out=s["out"])


# --------------------------------------------------------------------------- work, tolerance
def work(case):
    c = case
    kind = c["kind"]
    sz = 4 if c.get("dtype", "f32") == "f32" else 2
    if kind in ("linear", "lora"):
        T, m, n, q = c["T"], c["m"], c["n"], c["q"]
        nblk = _blocks(q, c["est"])
        nx = 1 if c["shared"] else nblk
        r = c["r"] if kind == "linear" else c["rl"] + min(c["r"], c["rl"])
        b = sz * (nx * T * n + m * n + nblk * T * m) + 4.0 * (r * (m + n) + q * r * r)
        f = 2.0 * (nx * T * m * n + nx * T * n * r + (q if nx == 1 else nblk) * T * r * m + q * m * r * r)
        if c.get("loss"):
            b += sz * T * m
            f += 3.0 * nblk * T * m
        return dict(bytes=b, flops=f)
    if kind == "attention":
        rows, dh, L = c["nblk"] * c["T"], c["dh"], c["seq"]
        return dict(bytes=2.0 * sz * rows * dh * (c["heads"] + c["kv_heads"]),
                    flops=rows / L * c["heads"] * 4.0 * dh * L * (L + 1) / 2)
    r = c["r"]
    if kind == "refresh":
        rows = sum(m + n for m, n in _opt_sides(c))
        return dict(bytes=8.0 * rows * r, flops=4.0 * rows * r * r)
    if kind == "update":
        b = f = 0.0
        for m, n in _opt_sides(c):
            b += 2.0 * sz * m * n + 4.0 * r * (m + n) + 4.0 * c["q"] * r * r + 16.0 * r * r
            f += 2.0 * m * n * r + 2.0 * m * r * r
        return dict(bytes=b, flops=f)
    nblk, T, L = 2 * c["q"], c["T"], c["seq"]
    b = 2.0 * sz * nblk * T * c["d"]
    f = nblk * T / L * 2.0 * c["d"] * L * (L + 1)
    for m, n in _layer_sides(c).values():
        b += sz * m * n + 4.0 * r * (m + n) + 4.0 * c["q"] * r * r
        f += 2.0 * nblk * T * (m * n + r * (m + n)) + 2.0 * c["q"] * m * r * r
    return dict(bytes=b, flops=f)


def tolerance(case):
    kind, dtype = case["kind"], case.get("dtype", "f32")
    if kind == "refresh":  # float64 inside, one rounding to fp32
        return dict(rel=1e-7, max=1e-5)
    if dtype == "f32":
        return dict(rel=5e-6, max=1e-4)
    if kind == "layer":  # stored activations round between the stages
        return dict(rel=2e-2, max=2e-1) if dtype == "bf16" else dict(rel=3e-3, max=3e-2)
    return dict(rel=7e-3, max=3e-2) if dtype == "bf16" else dict(rel=9e-4, max=4e-3)


# --------------------------------------------------------------------------- float64 reference
def _perturbed(mt, j, s):
    return mt["W"].double() + (s * EPS) * (mt["U"].double() @ mt["Z"][j].double() @ mt["V"].double().t())


def _attention(Q, K, V, seq, heads, kv_heads, dh):
    """Causal attention of rows x (heads dh) in float64, a few sequences at a time."""
    rows = Q.shape[0]
    out = torch.empty(rows, heads * dh, dtype=torch.float64, device=Q.device)
    mask = torch.ones(seq, seq, dtype=torch.bool, device=Q.device).triu_(1)
    step = max(1, int(2e8 // (heads * seq * seq)))
    for a in range(0, rows // seq, step):
        sl = slice(a * seq, min(rows, (a + step) * seq))
        cut = lambda t, h: t[sl].double().reshape(-1, seq, h, dh).transpose(1, 2).contiguous()  # noqa: E731
        q, k, v = cut(Q, heads), cut(K, kv_heads), cut(V, kv_heads)
        if kv_heads != heads:
            k = k.repeat_interleave(heads // kv_heads, 1)
            v = v.repeat_interleave(heads // kv_heads, 1)
        p = (q @ k.transpose(2, 3).contiguous()).div_(math.sqrt(dh)).masked_fill_(mask, -math.inf).softmax(-1)
        out[sl] = (p @ v).transpose(1, 2).reshape(-1, heads * dh)
    return out


def _rms(x, gamma):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-6) * gamma.double()


def _rope(x, seq, heads):
    dh = x.shape[1] // heads
    i = torch.arange(dh // 2, device=x.device, dtype=torch.float64)
    ang = torch.arange(seq, device=x.device, dtype=torch.float64)[:, None] * 10000.0 ** (-2.0 * i / dh)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]
    y = x.reshape(-1, seq, heads, dh)
    a, b = y[..., : dh // 2], y[..., dh // 2:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1).reshape(x.shape)


def exact(case, seed):
    c = dict(case)
    s = _inputs(c, seed)
    kind = c["kind"]
    if kind in ("linear", "lora"):
        T, m = c["T"], c["m"]
        bq, bs = _table(c["q"], c["est"])
        Y = torch.empty(len(bq) * T, m, dtype=torch.float64, device="cuda")
        for b, (j, sg) in enumerate(zip(bq, bs)):
            if kind == "linear":
                Wb = _perturbed(s, j, sg)
            else:
                d = {k: s[k].double() for k in LORA_KEYS}
                A = d["A"] + (sg * EPS) * (d["UA"] @ d["ZA"][j] @ d["VA"].t())
                B = d["B"] + (sg * EPS) * (d["UB"] @ d["ZB"][j] @ d["VB"].t())
                Wb = s["W"].double() + SCALE * (B @ A)
            x = s["X"] if c["shared"] else s["X"][b * T:(b + 1) * T]
            torch.mm(x.double(), Wb.t(), out=Y[b * T:(b + 1) * T])
        if kind == "linear" and c["loss"]:
            dev = Y.reshape(len(bq), T, m) - s["Ystar"].double()
            return Y, (0.5 / T) * dev.square_().sum((1, 2)) if c["dtype"] == "f32" else None
        return Y
    if kind == "attention":
        return _attention(s["Q"], s["K"], s["V"], c["seq"], c["heads"], c["kv_heads"], c["dh"])
    if kind == "refresh":
        out = []
        for om in s["omega"]:
            o = om.double().cpu()
            Q, R = torch.linalg.qr(o)
            out.append((Q * R.diagonal().sign()).cuda())
        return out
    if kind == "update":
        gv = s["g"].double()
        out = []
        for it in s["items"]:
            zb = (gv[:, None, None] * it["Z"].double()).mean(0)
            m1 = BETA1 * it["M1"].double() + (1 - BETA1) * zb
            m2 = BETA2 * it["M2"].double() + (1 - BETA2) * zb * zb
            S = (m1 / (1 - BETA1 ** STEP)) / ((m2 / (1 - BETA2 ** STEP)).sqrt() + EPS_ADAM)
            W = it["W"].double() - LR * (it["U"].double() @ S @ it["V"].double().t())
            out.append([W, m1, m2])
        return out
    bq, bs = _table(c["q"], "central")
    T = c["T"]
    heads, dh = c["heads"], c["d"] // c["heads"]
    out = torch.empty(len(bq) * T, c["d"], dtype=torch.float64, device="cuda")
    for b, (j, sg) in enumerate(zip(bq, bs)):
        W = lambda nm: _perturbed(s["mats"][nm], j, sg).t()  # noqa: E731
        H = s["H"][b * T:(b + 1) * T].double()
        A = _rms(H, s["norms"]["rms1_gamma"])
        C = _attention(_rope(A @ W("q"), c["seq"], heads), _rope(A @ W("k"), c["seq"], heads), A @ W("v"), c["seq"],
                       heads, heads, dh)
        H2 = H + C @ W("o")
        A2 = _rms(H2, s["norms"]["rms2_gamma"])
        out[b * T:(b + 1) * T] = H2 + (torch.nn.functional.silu(A2 @ W("gate")) * (A2 @ W("up"))) @ W("down")
    return out
