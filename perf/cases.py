"""The calls whose speed matters to a user of this library, with inputs drawn from a seed.

Layer shapes are Mamba-2's (head dimension 64, state 128, one or two B/C groups): 24, 32, 64 and 80 heads are the
130M, 350M, 1.3B and 2.7B widths (d_model = 32 * heads).  Kinds of case:

  scan      one SSD layer, forward + backward under sequence checkpoints (training)
  prefill   one SSD layer, forward only, no checkpoint kept
  decode    one SSD layer, the recurrence token by token on a kept state
  train     a residual stack of whole pre-norm blocks on the two-axis checkpoint grid, forward + backward
  prompt    the same stack, forward only from an empty state: reading a prompt
  generate  the same stack, one token for each of `nseq` sequences on kept states
"""
import math

import torch

import paper_2411_19460_amd as pk

P, N = 64, 128                 # head dimension and state of every bf16 case
HEADS = (24, 32, 64, 80)


def listed():
    return [
        # one token of one 2.7B-shaped layer: the smallest call there is, a single launch
        dict(name="decode-2.7b", kind="decode", batch=1, tokens=1, heads=80, groups=1),
        # the fp32 configuration of the benchmark list: a handful of tiny launches
        dict(name="scan-f32-tiny", kind="scan", dtype="f32", batch=1, tokens=512, heads=4, headdim=16, state=16, groups=1,
             chunk=64, segment=256, packed=False, states=False, autograd=False),
        # a layer of the 130M model checked or trained in fp32 on a short, ragged sequence
        dict(name="scan-f32-130m", kind="scan", dtype="f32", batch=1, tokens=1999, heads=24, headdim=P, state=N, groups=1,
             chunk=256, segment=1024, packed=False, states=True, autograd=False),
        # the 130M layer of the benchmark list
        dict(name="scan-130m-8k", kind="scan", dtype="bf16", batch=1, tokens=8192, heads=24, headdim=P, state=N, groups=1,
             chunk=256, segment=2048, packed=False, states=False, autograd=False),
        # a batch of packed sequences of odd length through the differentiable face, states in and out
        dict(name="scan-350m-packed", kind="scan", dtype="bf16", batch=2, tokens=3001, heads=32, headdim=P, state=N, groups=2,
             chunk=128, segment=1024, packed=True, states=True, autograd=True),
        # the headline configuration of the benchmark
        dict(name="scan-2.7b-64k", kind="scan", dtype="bf16", batch=1, tokens=65536, heads=80, headdim=P, state=N, groups=1,
             chunk=256, segment=4096, packed=False, states=False, autograd=False),
        # video-scale training of one layer
        dict(name="scan-2.7b-256k", kind="scan", dtype="bf16", batch=1, tokens=262144, heads=80, headdim=P, state=N, groups=1,
             chunk=256, segment=16384, packed=False, states=False, autograd=False),
        # a prompt of odd length through one layer
        dict(name="prefill-2.7b", kind="prefill", batch=1, tokens=10007, heads=80, groups=1, chunk=256, segment=4096),
        # training step of whole blocks at the 2.7B width, two layer inputs kept, four segments
        dict(name="train-2.7b", kind="train", layers=2, tokens=16384, heads=80, groups=1, chunk=256, segment=4096, interval=1),
        # a prompt of odd length through four 2.7B blocks
        dict(name="prompt-2.7b", kind="prompt", layers=4, tokens=6001, heads=80, groups=1, chunk=256, segment=4096),
        # a token for one sequence, and for a full serving batch, through eight 2.7B blocks
        dict(name="generate-2.7b-1", kind="generate", layers=8, nseq=1, heads=80, groups=1),
        dict(name="generate-2.7b-16", kind="generate", layers=8, nseq=16, heads=80, groups=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("scan", "scan", "scan-f32", "prefill", "decode", "train", "prompt", "generate"))
    heads, groups = rng.choice(HEADS), rng.choice((1, 1, 1, 2))
    if kind == "scan":
        batch = rng.choice((1, 1, 2, 4))
        tokens = _log(rng, 512, 262144 * 80 // (heads * batch) if heads * batch > 80 else 262144)
        return dict(kind=kind, dtype="bf16", batch=batch, tokens=tokens, heads=heads, headdim=P, state=N, groups=groups,
                    chunk=rng.choice((128, 256, 256)), segment=rng.choice((1024, 2048, 4096, 8192, 16384)),
                    packed=rng.random() < 0.25, states=rng.random() < 0.5, autograd=rng.random() < 0.25)
    if kind == "scan-f32":
        return dict(kind="scan", dtype="f32", batch=rng.choice((1, 2)), tokens=_log(rng, 256, 4096), heads=4 * rng.randint(1, 6),
                    headdim=rng.choice((16, 32, 64)), state=rng.choice((16, 64, 128)), groups=groups,
                    chunk=rng.choice((64, 128, 256)), segment=rng.choice((256, 1024)), packed=rng.random() < 0.25,
                    states=rng.random() < 0.5, autograd=rng.random() < 0.25)
    if kind == "prefill":
        return dict(kind=kind, batch=rng.choice((1, 1, 2)), tokens=_log(rng, 300, 131072), heads=heads, groups=groups, chunk=256,
                    segment=rng.choice((2048, 4096, 16384)))
    if kind == "decode":
        return dict(kind=kind, batch=_log(rng, 1, 64), tokens=rng.choice((1, 1, 1, 2, 4)), heads=heads, groups=groups)
    size = (heads / 80) ** 2            # a block's products grow with the square of the width
    if kind == "train":
        layers = rng.randint(1, 4)
        return dict(kind=kind, layers=layers, tokens=_log(rng, 1024, min(65536, int(2 * 16384 / (layers * size)))), heads=heads,
                    groups=groups, chunk=256, segment=rng.choice((1024, 2048, 4096)), interval=rng.randint(1, layers))
    if kind == "prompt":
        layers = rng.randint(1, 8)
        return dict(kind=kind, layers=layers, tokens=_log(rng, 200, min(65536, int(4 * 24576 / (layers * size)))), heads=heads,
                    groups=groups, chunk=256, segment=rng.choice((2048, 4096)))
    return dict(kind=kind, layers=rng.randint(2, 12), nseq=rng.randint(1, 16), heads=heads, groups=groups)


# ---- inputs ----------------------------------------------------------------------------------------------------------------

def _scan_inputs(g, dtype, Bt, L, H, hd, n, G):
    """The value distributions of the benchmark's layers: dt in [9e-4, 0.096], A in [-16, -1], B and C scaled by the state."""
    dev = g.device
    normal = lambda *shape: torch.randn(shape, generator=g, device=dev, dtype=dtype)  # noqa: E731
    x = normal(Bt, L, H, hd)
    dt = torch.nn.functional.softplus(torch.rand((Bt, L, H), generator=g, device=dev) * 4.7 - 7.0).to(dtype)
    A = -torch.exp(torch.rand(H, generator=g, device=dev) * math.log(16.0))
    B, C = (normal(Bt, L, G, n) / math.sqrt(n) for _ in range(2))
    D = torch.randn(H, generator=g, device=dev)
    return [x, dt, A, B, C, D]


def _layers(g, nlayers, H, G):
    """Random-init blocks: projections scaled by their fan-in, step-size bias from [1e-3, 0.1], norm weights around 1."""
    dev, dm, di = g.device, 32 * H, H * P
    conv, d_in = di + 2 * G * N, 2 * di + 2 * G * N + H
    normal = lambda *shape, dtype=torch.float32: torch.randn(shape, generator=g, device=dev, dtype=dtype)  # noqa: E731
    out = []
    for _ in range(nlayers):
        step = torch.exp(torch.rand(H, generator=g, device=dev) * math.log(100.0) + math.log(1e-3))
        out.append({
            "W_in": normal(d_in, dm, dtype=torch.bfloat16).mul_(dm ** -0.5), "conv_w": normal(conv, 4) * 0.5, "conv_b": normal(conv) * 0.2,
            "dt_bias": step + torch.log(-torch.expm1(-step)), "A": -torch.exp(torch.rand(H, generator=g, device=dev) * math.log(16.0)),
            "D": normal(H), "norm_w": 1.0 + 0.3 * normal(di), "W_out": normal(dm, di, dtype=torch.bfloat16).mul_(di ** -0.5),
            "pre_norm_w": 1.0 + 0.3 * normal(dm)})
    return out


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    c, kind, H, G = case, case["kind"], case["heads"], case["groups"]
    s = {"case": c}
    if kind in ("scan", "prefill", "decode"):
        dtype = torch.float32 if c.get("dtype") == "f32" else torch.bfloat16
        Bt, L, hd, n = c["batch"], c["tokens"], c.get("headdim", P), c.get("state", N)
        s["in"] = _scan_inputs(g, dtype, Bt, L, H, hd, n, G)
        x, _, _, B = s["in"][:4]
        state = lambda: torch.randn((Bt, H, hd, n), generator=g, device=dev)  # noqa: E731
        if kind == "decode":
            s["state"], s["y"] = state(), torch.empty_like(x)
        else:
            shape = pk.make_shape(x, B, c["chunk"], c["segment"])
            space = lambda back: torch.empty(pk.binding.ssd_workspace_bytes(shape, back), dtype=torch.uint8, device=dev)  # noqa: E731
        if kind == "prefill":
            s["ws"], s["out"] = space(False), {"y": torch.empty_like(x), "final_state": torch.empty((Bt, H, hd, n), device=dev)}
        if kind == "scan":
            s["dy"] = torch.randn(x.shape, generator=g, device=dev, dtype=dtype)
            s["init"], s["dfinal"] = (state(), state()) if c["states"] else (None, None)
            s["reset"] = None
            if c["packed"]:          # sequences of about 700 tokens, one behind the other
                s["reset"] = (torch.rand((Bt, L), generator=g, device=dev) < 1 / 700).to(torch.uint8)
                s["reset"][:, 0] = 1
            if c["autograd"]:
                s["in"] = [t.requires_grad_() for t in s["in"]]
                s["init"] = None if s["init"] is None else s["init"].requires_grad_()
            else:                    # a training loop keeps its scratch, its outputs and its gradients
                s["ws"], s["ws_back"] = space(False), space(True)
                s["dA"], s["dD"] = (torch.empty(H, device=dev) for _ in range(2))
                new = torch.empty_like
                s["out"] = {"y": new(x), "final_state": torch.empty((Bt, H, hd, n), device=dev),
                            "boundary_states": torch.empty((Bt, -(-L // c["segment"]), H, hd, n), device=dev)}
                s["grads"] = {"dx": new(x), "ddt": new(s["in"][1]), "dB": new(B), "dC": new(B), "dinit_state": torch.empty((Bt, H, hd, n), device=dev)}
        return s
    s["layers"] = _layers(g, c["layers"], H, G)
    rows = c["nseq"] if kind == "generate" else c["tokens"]
    s["x"] = torch.randn((rows, 32 * H), generator=g, device=dev, dtype=torch.bfloat16)
    if kind == "train":
        s["dout"] = torch.randn(s["x"].shape, generator=g, device=dev, dtype=torch.bfloat16)
    if kind == "generate":           # the states behind some prompt; the first call's scratch is handed to the next
        lead = (rows, c["layers"]) if rows > 1 else (c["layers"],)
        s["ssm"] = torch.randn(lead + (H, P, N), generator=g, device=dev) * 0.3
        s["conv"] = torch.randn(lead + (3, H * P + 2 * G * N), generator=g, device=dev, dtype=torch.bfloat16)
        s["out"], s["ws"] = torch.empty_like(s["x"]), None
    return s


# ---- one pass --------------------------------------------------------------------------------------------------------------

def run(s):
    c, kind, H, G = s["case"], s["case"]["kind"], s["case"]["heads"], s["case"]["groups"]
    if kind == "decode":
        return pk.ssd_decode(*s["in"], s["state"], out=s["y"]), s["state"]
    if kind == "prefill":
        y, final, _ = pk.ssd_fwd(*s["in"], c["chunk"], c["segment"], workspace=s["ws"], out=s["out"], want_boundary=False)
        return y, final
    if kind == "scan" and c["autograd"]:
        y, final = pk.ssd_scan(*s["in"], c["chunk"], c["segment"], s["init"], 0, s["reset"])
        wrt = s["in"] + ([] if s["init"] is None else [s["init"]])
        ends = ([y], [s["dy"]]) if s["dfinal"] is None else ([y, final], [s["dy"], s["dfinal"]])
        return [y.detach(), final.detach()] + list(torch.autograd.grad(ends[0], wrt, ends[1]))
    if kind == "scan":
        y, final, bnd = pk.ssd_fwd(*s["in"], c["chunk"], c["segment"], s["init"], workspace=s["ws"], out=s["out"], seq_reset=s["reset"])
        grads = pk.ssd_bwd(*s["in"], s["dy"], c["chunk"], c["segment"], s["init"], s["dfinal"], bnd, workspace=s["ws_back"],
                           dA=s["dA"], dD=s["dD"], out=s["grads"], seq_reset=s["reset"])
        return {"y": y, "final_state": final, "boundary_states": bnd, **grads}
    model = (s["layers"], H, P, G, N)
    if kind == "train":
        f = pk.magc_blockstack_fwd(s["x"], *model, c["chunk"], c["segment"], c["interval"])
        b = pk.magc_blockstack_bwd(s["x"], s["layers"], s["dout"], f["l_ckpt"], f["ssm_ckpt"], f["conv_ckpt"], *model[1:],
                                   c["chunk"], c["segment"], c["interval"])
        return {"out": f["out"], "dx0": b["dx0"], "grads": b["grads"]}
    if kind == "prompt":
        r = pk.magc_blockstack_infer(s["x"], *model, c["chunk"], c["segment"])
    elif c["nseq"] == 1:
        r = pk.magc_blockstack_infer(s["x"], *model, 256, 4096, ssm_state=s["ssm"], conv_state=s["conv"], out=s["out"], workspace=s["ws"])
        s["ws"] = r["workspace"]
    else:
        r = pk.magc_blockstack_decode(s["x"], *model, 256, 4096, s["ssm"], s["conv"], out=s["out"], workspace=s["ws"])
        s["ws"] = r["workspace"]
        return r["out"], s["ssm"], s["conv"]
    return r["out"], r["ssm_state"], r["conv_state"]


# ---- what a pass cannot do without -----------------------------------------------------------------------------------------

def work(case):
    """Inputs read once, outputs written once; the contractions of the recurrence (two per token, head, channel and state
    element forward, four backward) and of the projections (one forward, two backward).  What the checkpoint grid recomputes
    is not counted."""
    c, kind, H, G = case, case["kind"], case["heads"], case["groups"]
    hd, n = c.get("headdim", P), c.get("state", N)
    if kind in ("scan", "prefill", "decode"):
        e = 4 if c.get("dtype") == "f32" else 2
        T, state = c["batch"] * c["tokens"], c["batch"] * H * hd * n * 4
        X, dt, bc = T * H * hd * e, T * H * e, T * G * n * e
        byte, flop = 2 * X + dt + 2 * bc, 4 * n * hd * H * T         # x, dt, B, C -> y
        if kind == "decode":
            byte += 2 * state
        elif kind == "prefill":
            byte += state
        else:                                                        # dy -> dx, ddt, dB, dC; final, boundary and initial states
            byte += 2 * X + dt + 2 * bc + state * (2 + -(-c["tokens"] // c["segment"]) + (2 if c["states"] else 0))
            flop *= 3
        return {"bytes": byte, "flops": flop}
    dm, di, gn = 32 * H, H * P, G * N
    weights = (2 * di + 2 * gn + H) * dm + dm * di
    small = 5 * (di + 2 * gn) + di + dm + 3 * H                      # fp32 parameters
    states = c["layers"] * (di * N * 4 + 3 * (di + 2 * gn) * 2)      # of one sequence
    T = c["nseq"] if kind == "generate" else c["tokens"]
    byte = c["layers"] * (weights * 2 + small * 4) + 2 * T * dm * 2
    flop = T * c["layers"] * (2 * weights + 4 * N * di + 8 * (di + 2 * gn))
    if kind == "generate":
        byte += 2 * T * states
    elif kind == "prompt":
        byte += states
    else:                                                            # dout -> dx0 and the fp32 parameter gradients
        byte += 2 * T * dm * 2 + c["layers"] * (weights + small) * 4
        flop *= 3
    return {"bytes": byte, "flops": flop}


def tolerance(case):
    """What two correct implementations differ by (measured between chunk lengths and kernel families, with a margin)."""
    if case.get("dtype") == "f32":
        return {"rel": 1e-5}         # 32-bit sums
    if case["kind"] == "decode":
        return {"rel": 4e-3}         # one bf16 rounding of y, fp32 states
    if case["kind"] in ("scan", "prefill"):
        return {"rel": 1e-2}         # bf16 operands, fp32 accumulation
    # every layer rounds its activations to bf16 on top of what the layers before it did: a random walk over the layers; the
    # parameter gradients of a training step pass through two such walks
    return {"rel": (1.5e-2 if case["kind"] == "train" else 1e-2) * math.sqrt(max(1, case["layers"] * (1 if case["kind"] == "train" else 0.5)))}
