"""Performance cases of the NOBLE linear layer: what its users run, from one decoded token to a training step of
32768 tokens, through the public entry points of ``paper_2603_06492_amd.noble``.

Every case is one layer.  ``mode`` names the entry point:

* ``serve``:  ``noble_linear_fwd_static``, the forward of a loop that may not allocate (y and the parameters kept);
* ``infer``:  the ``NobleLinear`` module under ``torch.no_grad()``;
* ``train``:  ``noble_linear_fwd`` + ``noble_linear_bwd`` with a workspace and gradient buffers that the program keeps;
* ``module``: ``NobleLinear`` forward and autograd backward, gradients set to None in between.
"""

import math

import torch

from paper_2603_06492_amd import noble

DTYPES = {"bf16": (torch.bfloat16, noble.NOBLE_BF16), "f32": (torch.float32, noble.NOBLE_F32)}
PARAMS = ("W", "b", "W_down", "omega1", "phi1", "M", "omega2", "phi2", "W_up")
STORAGE = ("W", "W_down", "M", "W_up")
LARGEST = 2 * 32768 * (2048 * 8192 + 128 * (2048 + 8192) + 128 * 128) * 3   # flops of the largest listed case


def _case(name, mode, T, d_in, d_out, r, dtype="bf16", activation="cosnet", groups=1):
    return dict(name=name, mode=mode, T=T, d_in=d_in, d_out=d_out, r=r, dtype=dtype, activation=activation,
                groups=groups)


def listed():
    return [
        # one token of one sequence: the grouped Q, K and V of a 1.5B block in a decode loop that may not allocate
        _case("decode1_qkv", "serve", 1, 2048, 6144, 128, groups=3),
        # one token of each of 16 sequences: the 1.5B FFN's up-projection in batched decoding
        _case("decode16_ffn_up", "infer", 16, 2048, 8192, 128),
        # prefill of one prompt of an odd length: the 1.5B FFN's down-projection
        _case("prefill_ffn_down", "infer", 777, 8192, 2048, 128),
        # a ViT-B layer over a small batch of images (8 x 197 tokens), classified without gradients
        _case("vit_images_up", "infer", 8 * 197, 768, 3072, 32),
        # the 250M model's QKV layer in a training loop written with the module: 8 x 1024 tokens per GPU
        _case("train_250m_qkv", "module", 8192, 1024, 3072, 64),
        # ViT-B training, 128 images x 197 tokens: the FFN's down-projection
        _case("train_vitb_down", "train", 128 * 197, 3072, 768, 32),
        # the 1.5B model's attention output projection: 8 x 1024 tokens per GPU
        _case("train_1p5b_o", "train", 8192, 2048, 2048, 128),
        # the largest rank of the ablation, an activation variant, a short batch: fine-tuning on 4 x 500 tokens
        _case("finetune_r256_gelu", "module", 2000, 2048, 2048, 256, activation="gelu_m"),
        # four-block 1.5B stack, 16 x 2048 tokens: Q, K and V of a block as one grouped call
        _case("train_stack_qkv", "train", 32768, 2048, 6144, 128, groups=3),
        # the same stack's FFN up-projection, the largest layer of the benchmark
        _case("train_stack_ffn_up", "train", 32768, 2048, 8192, 128),
        # the float32 path at its smallest, a training step of a toy layer: launches and host work
        _case("tiny_f32", "module", 256, 64, 64, 8, dtype="f32"),
        # the float32 path on a real layer: reference runs and small-model training in full precision
        _case("train_f32_768", "train", 2048, 768, 768, 32, dtype="f32"),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges: serving of 1 to 2048 tokens, bf16 training of 256 to 32768 tokens,
    float32 training of 64 to 4096 tokens; widths that are multiples of 8 (of 8 x groups for d_out)."""
    while True:
        kind = rng.choice(("serve", "infer", "infer", "train", "train", "module", "f32"))
        f32 = kind == "f32"
        activation = rng.choice(("cosnet",) * 6 + ("cosnet3", "gelu_m", "tanh", "cos"))
        groups = rng.choice((1, 1, 1, 3))
        if f32:
            mode, T = rng.choice(("train", "module")), _spread(rng, 64, 4096)
            lo, hi, ranks = 64, 1024, (8, 16, 32, 64)
        else:
            mode = kind
            T = _spread(rng, 1, 2048) if kind in ("serve", "infer") else _spread(rng, 256, 32768)
            lo, hi, ranks = 512, 8192, (32, 64, 128, 128, 256)
        r = rng.choice(ranks)
        if activation == "cosnet3":
            r = min(r, 128)
        d_in = 8 * _spread(rng, lo // 8, hi // 8)
        d_out = 8 * groups * max(1, _spread(rng, lo // 8, hi // 8) // groups)
        if rng.random() < 0.5:   # the usual widths are multiples of 128 (64 for the smallest)
            q = 64 if f32 else 128
            d_in, d_out = max(q, d_in // q * q), max(q * groups, d_out // (q * groups) * q * groups)
        c = _case("", mode, T, d_in, d_out, r, "f32" if f32 else "bf16", activation, groups)
        del c["name"]
        if work(c)["flops"] <= LARGEST:
            return c


def _shapes(c):
    G, r, L = c["groups"], c["r"], noble.layers(c["activation"])
    R = G * r
    M = (r, r) if G == 1 else (G, r, r)
    v2 = (R,)
    if L == 3:
        M, v2 = (2,) + M, (2, R)
    s = dict(W=(c["d_in"], c["d_out"]), b=(c["d_out"],), W_down=(c["d_in"], R), omega1=(R,), phi1=(R,), M=M,
             omega2=v2, phi2=v2, W_up=(R, c["d_out"] // G))
    if L == 1:
        s.update(M=None, omega2=None, phi2=None)
    return s


def _inputs(c, seed):
    """x, dy and the parameters: standard normal activations, weights of variance 1 / fan-in, frequencies around one
    and phases over the whole period, so that the branch contributes as it does in a trained layer."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    sd = DTYPES[c["dtype"]][0]

    def normal(shape, std, dt):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(dt)

    t = {"x": normal((c["T"], c["d_in"]), 1.0, sd), "dy": normal((c["T"], c["d_out"]), 1.0, sd)}
    std = {"W": c["d_in"] ** -0.5, "W_down": c["d_in"] ** -0.5, "M": c["r"] ** -0.5, "W_up": c["r"] ** -0.5}
    for n, shape in _shapes(c).items():
        if shape is None:
            t[n] = None
        elif n in STORAGE:
            t[n] = normal(shape, std[n], sd)
        elif n.startswith("omega"):
            t[n] = 1.0 + normal(shape, 0.1, torch.float32)
        elif n.startswith("phi"):
            t[n] = torch.rand(shape, generator=g, device="cuda") * (2.0 * math.pi)
        else:
            t[n] = normal(shape, 0.1, torch.float32)
    return t


def prepare(case, seed):
    c, t = case, _inputs(case, seed)
    s = {"case": c}
    sd, code = DTYPES[c["dtype"]]
    if c["mode"] in ("infer", "module"):
        layer = noble.NobleLinear(c["d_in"], c["d_out"], c["r"], dtype=sd, activation=c["activation"],
                                  groups=c["groups"])
        with torch.no_grad():
            for n in PARAMS:
                if t[n] is not None:
                    getattr(layer, n).copy_(t[n])
        s.update(layer=layer, x=t["x"])
        if c["mode"] == "module":
            s["x"].requires_grad_(True)
            s["dy"] = t["dy"]
        return s
    s["in"] = [t["x"]] + [t[n] for n in PARAMS]
    s["y"] = torch.empty((c["T"], c["d_out"]), dtype=sd, device="cuda")
    if c["mode"] == "train":
        s["dy"] = t["dy"]
        s["reserve"], s["scratch"] = noble.alloc_workspace(c["T"], c["d_in"], c["d_out"], c["r"], code,
                                                           groups=c["groups"], activation=c["activation"])
        s["dx"] = torch.empty_like(t["x"])
        s["grads"] = {n: None if sh is None else torch.empty(sh, device="cuda") for n, sh in _shapes(c).items()}
    return s


def run(state):
    c = state["case"]
    mode = c["mode"]
    kw = dict(activation=c["activation"], groups=c["groups"])
    if mode == "serve":
        noble.noble_linear_fwd_static(*state["in"], state["y"], None, **kw)
        return {"y": state["y"]}
    if mode == "infer":
        with torch.no_grad():
            return {"y": state["layer"](state["x"])}
    if mode == "module":
        layer, x = state["layer"], state["x"]
        layer.zero_grad(set_to_none=True)
        x.grad = None
        y = layer(x)
        y.backward(state["dy"])
        out = {"y": y.detach(), "dx": x.grad}
        out.update({"d" + n: p.grad for n, p in layer.named_parameters()})
        return out
    x, W, b, *branch = state["in"]
    noble.noble_linear_fwd(x, W, b, *branch, state["y"], state["reserve"], state["scratch"], **kw)
    g = state["grads"]
    noble.noble_linear_bwd(state["dy"], x, W, *branch, state["reserve"], state["dx"], g["W"], g["b"], g["W_down"],
                           g["M"], g["W_up"], g["omega1"], g["phi1"], g["omega2"], g["phi2"], state["scratch"], **kw)
    out = {"y": state["y"], "dx": state["dx"]}
    out.update({"d" + n: t for n, t in g.items() if t is not None})
    return out


def work(case):
    c = case
    T, di, do, G, r = c["T"], c["d_in"], c["d_out"], c["groups"], c["r"]
    es = 2 if c["dtype"] == "bf16" else 4
    n = {k: math.prod(s) for k, s in _shapes(c).items() if s is not None}
    mix = noble.layers(c["activation"]) - 1
    flops = 2.0 * T * (di * do + G * r * di + r * do + mix * G * r * r)
    params = sum(v * (es if k in STORAGE else 4) for k, v in n.items())
    nbytes = T * (di + do) * es + params
    if c["mode"] in ("train", "module"):
        flops *= 3
        nbytes += T * (di + do) * es                                                # dy and dx
        nbytes += params if c["mode"] == "module" else sum(n.values()) * 4          # the gradients
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(case):
    # bf16: the rounding of the 16-bit results and of the products' operands; float32: sums over d_in, d_out and T
    # in another order, and the hardware's sine and cosine
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 1e-5, "max": 4e-4}


def _f(activation):
    name = activation[:-2] if activation.endswith("_m") else activation
    return {"tanh": torch.tanh, "gelu": torch.nn.functional.gelu,
            "leaky_relu": torch.nn.functional.leaky_relu}.get(name, torch.cos)


def exact(case, seed):
    """The layer in float64, its gradients by torch's autograd."""
    c, t = case, _inputs(case, seed)
    grad = c["mode"] in ("train", "module")
    t = {n: None if v is None else v.double().requires_grad_(grad and n != "dy") for n, v in t.items()}
    G, r, L, f = c["groups"], c["r"], noble.layers(c["activation"]), _f(c["activation"])
    dog = c["d_out"] // G
    Ms = [] if L == 1 else [t["M"]] if L == 2 else [t["M"][0], t["M"][1]]
    vec = [] if L == 1 else [(t["omega2"], t["phi2"])] if L == 2 else [(t["omega2"][i], t["phi2"][i]) for i in (0, 1)]
    H = t["x"] @ t["W_down"]
    parts = []
    for g in range(G):
        s = slice(g * r, (g + 1) * r)
        C = f(H[:, s] * t["omega1"][s] + t["phi1"][s])
        for M, (w, p) in zip(Ms, vec):
            C = f((C @ (M if G == 1 else M[g])) * w[s] + p[s])
        parts.append(C @ t["W_up"][s])
    y = t["x"] @ t["W"] + t["b"] + (parts[0] if G == 1 else torch.cat(parts, 1))
    assert y.shape[1] == G * dog
    if not grad:
        return {"y": y}
    names = ["x"] + [n for n in PARAMS if t[n] is not None]
    grads = torch.autograd.grad(y, [t[n] for n in names], t["dy"])
    return {"y": y.detach(), **{"d" + n: v for n, v in zip(names, grads)}}
