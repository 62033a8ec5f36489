"""Performance cases of the region-reuse denoising step.

Each case is one call that an editing program makes through the package's
public entry points, at the sizes of the benchmark and the tests: 512, 1024
and 2048 px latents (32, 64 and 128 patches a side), 10-20 % of the tokens
active in an edit, PixArt-alpha's widths (hidden 1152, 16 heads of 72, MLP
4608, 120 text tokens of 4096 features).  Weights are random with the
statistics of a model whose branches matter: query and key projections three
times the N(0, 0.02) of the others (attention logits of standard deviation
about 4) and residual gates near 1.  Cached keys and values have the standard
deviation that such projections produce.

Whole steps have 28 blocks; the other step cases have a few, which is enough
that their weights are not in a cache from one pass to the next (several
states are run in turn), and short enough that a change of rounding in one
block does not travel far.
"""
import math
import types

import numpy as np
import torch

from paper_2608_29809_amd.runtime import ActiveSet, RegionCacheModel, maps_from_logits

C, HEADS, D, F, M, TEXT = 1152, 16, 72, 4608, 120, 4096
MATS = {"qkv_w": (3 * C, C), "proj_w": (C, C), "xq_w": (C, C), "xkv_w": (2 * C, C), "xproj_w": (C, C),
        "fc1_w": (F, C), "fc2_w": (C, F)}
VECS = {"qkv_b": (3 * C,), "proj_b": (C,), "xq_b": (C,), "xkv_b": (2 * C,), "xproj_b": (C,), "fc1_b": (F,),
        "fc2_b": (C,), "sst": (6, C)}
GLOBALS = {"pe_w": (C, 16), "pe_b": (C,), "temb_w1": (C, 256), "temb_b1": (C,), "temb_w2": (C, C), "temb_b2": (C,),
           "tblock_w": (6 * C, C), "tblock_b": (6 * C,), "cap_w1": (C, TEXT), "cap_b1": (C,), "cap_w2": (C, C),
           "cap_b2": (C,), "fin_w": (32, C), "fin_b": (32,), "fin_sst": (2, C)}
GLOBAL_MATS = ("pe_w", "temb_w1", "temb_w2", "tblock_w", "cap_w1", "cap_w2", "fin_w")
T_NOW, T_NEXT = 789, 736  # consecutive entries of the 20-step sampling grid
GUIDANCE = 4.5


def _step(kind, gh, gw, layers, frac=0.0, batch=1, dtype="bf16", latent=False, guided=False, padded=False, n_delta=0):
    return dict(kind=kind, gh=gh, gw=gw, layers=layers, frac=frac, batch=batch, dtype=dtype, latent=latent,
                guided=guided, padded=padded, n_delta=n_delta)


def listed():
    def case(name, c):
        c["name"] = name
        return c

    return [
        # the edit region read out of the aggregated maps at 1024 px: once a turn, its host waits for the counts
        case("localize_1024", dict(kind="localize", gh=64, gw=64, batch=1, n_delta=6, radius=1)),
        # the maps themselves from logits that a program kept: all blocks and heads at 1024 px
        case("maps_1024", dict(kind="maps", gh=64, gw=64, layers=28, n_delta=6)),
        # the prompt of a turn: caption projection and every block's text keys and values, one chain
        case("text", dict(kind="text", layers=28, batch=1, dtype="bf16")),
        # whole region step of a 512 px edit (15 %): few rows, the interactive case
        case("reuse_512", _step("reuse", 32, 32, 28, frac=0.15, latent=True)),
        # whole region step of a 1024 px edit, 723 active tokens: the benchmark's step
        case("reuse_1024", _step("reuse", 64, 64, 28, frac=0.1765, latent=True)),
        # blocks of a 2048 px edit (15 %): attention over 16384 keys
        case("reuse_2048", _step("reuse", 128, 128, 4, frac=0.15)),
        # a served batch: two images with guidance (four chains) and padded prompts at 10 %
        case("reuse_1024_guided", _step("reuse", 64, 64, 4, frac=0.10, batch=4, latent=True, guided=True, padded=True)),
        # the last dense step of a 512 px turn, whose attention maps localise the region
        case("dense_512_maps", _step("dense", 32, 32, 4, n_delta=5)),
        # blocks of the dense step that fills the cache at 1024 px
        case("dense_1024", _step("dense", 64, 64, 4)),
        # the same at 2048 px, the largest grid
        case("dense_2048", _step("dense", 128, 128, 2)),
        # a pool too large for the device: the slot stays in pinned host memory
        case("hosted_1024", _step("hosted", 64, 64, 4, frac=0.1765)),
        # single precision storage, as a program checks or debugs an edit with
        case("reuse_512_f32", _step("reuse", 32, 32, 4, frac=0.15, dtype="f32")),
    ]


def _grid(rng, lo, hi):
    """A patch grid of the aspect ratios that images come in, lo .. hi tokens, a multiple of 64 of them."""
    while True:
        n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        a = math.exp(rng.uniform(-0.6, 0.6))
        gh, gw = round(math.sqrt(n * a)), round(math.sqrt(n / a))
        gw += -gw % (64 // math.gcd(64, gh))
        if lo <= gh * gw <= hi and 0.4 < gh / gw < 2.5:
            return gh, gw


def draw(rng):
    kind = rng.choice(["localize", "maps", "text", "reuse", "reuse", "reuse", "reuse", "dense", "dense", "hosted"])
    if kind == "localize":
        gh, gw = _grid(rng, 256, 16384)
        return dict(kind=kind, gh=gh, gw=gw, batch=rng.randint(1, 6), n_delta=rng.randint(1, 8),
                    radius=rng.randint(0, 2))
    if kind == "maps":
        gh, gw = _grid(rng, 256, 8192)
        return dict(kind=kind, gh=gh, gw=gw, layers=rng.randint(4, 28), n_delta=rng.randint(1, 8))
    if kind == "text":
        return dict(kind=kind, layers=rng.randint(4, 28), batch=rng.randint(1, 6), dtype=rng.choice(["bf16", "bf16", "f32"]))
    dtype = "f32" if kind == "reuse" and rng.random() < 0.2 else "bf16"
    gh, gw = _grid(rng, 256, 16384 if kind == "reuse" and dtype == "bf16" else 8192 if kind == "dense" else 4096)
    frac = 0.0 if kind == "dense" else math.exp(rng.uniform(math.log(0.02), math.log(0.5)))
    big = gh * gw >= 8192
    batch = 1 if big else rng.choice([1, 1, 2, 3, 4])
    latent = rng.random() < 0.5
    return _step(kind, gh, gw, rng.randint(2, 3 if big else 5), frac=round(frac, 4), batch=batch, dtype=dtype, latent=latent,
                 guided=latent and batch % 2 == 0 and rng.random() < 0.5, padded=rng.random() < 0.3,
                 n_delta=rng.choice([0, 0, rng.randint(1, 8)]))


# ------------------------------------------------------------------ inputs

def _shape(case):
    return types.SimpleNamespace(
        hidden=C, heads=HEADS, head_dim=D, mlp=F, layers=case.get("layers", 1), text_len=M,
        text_dim=TEXT if case.get("latent", case["kind"] in ("text", "localize")) else C, grid_h=case.get("gh", 32),
        grid_w=case.get("gw", 32), latent_ch=4, patch=2, out_ch=8, dtype=case.get("dtype", "bf16"),
        token_mode=not case.get("latent", case["kind"] in ("text", "localize")))


def _weights(case, seed, token_mode):
    """Random weights as the model takes them (float32 arrays).  Every array is a window of one long stream of
    normals at a place of its own, which is much faster to make than a stream for each."""
    rng = np.random.default_rng([int(seed), 1])
    pool = rng.standard_normal(1 << 23, dtype=np.float32)
    pool *= np.float32(0.02)

    def take(shape):
        n = int(np.prod(shape))
        at = int(rng.integers(0, pool.size - n))
        return pool[at:at + n].reshape(shape)

    layers = []
    for _ in range(case["layers"]):
        lw = {k: take(s) for k, s in {**MATS, **VECS}.items()}
        for k, rows in (("qkv_w", 2 * C), ("xq_w", C), ("xkv_w", C)):
            lw[k] = lw[k].copy()
            lw[k][:rows] *= 3.0
        lw["sst"] = lw["sst"].copy()
        lw["sst"][[2, 5]] += 1.0
        layers.append(lw)
    w = {k: take(s) for k, s in GLOBALS.items() if not token_mode or k in ("tblock_w", "tblock_b")}
    w["layers"] = layers
    return w


def _regions(case, seed):
    """Per chain, the active tokens of an edit: those inside one to three ellipses, frac of the grid (guided pairs
    share theirs; chains differ in size by up to a third)."""
    rng = np.random.default_rng([int(seed), 2])
    gh, gw = case["gh"], case["gw"]
    yy, xx = np.meshgrid(np.arange(gh), np.arange(gw), indexing="ij")
    out = []
    for b in range(case["batch"]):
        if case["guided"] and b % 2:
            out.append(out[-1])
            continue
        field = np.full((gh, gw), -np.inf)
        for _ in range(int(rng.integers(1, 4))):
            cy, cx = rng.uniform(0.15, 0.85, 2) * (gh, gw)
            ry, rx = rng.uniform(0.08, 0.25, 2) * (gh, gw)
            field = np.maximum(field, -((yy - cy) / ry) ** 2 - ((xx - cx) / rx) ** 2)
        n = max(1, round(case["frac"] * gh * gw * (1.0 if case["batch"] == 1 else 1.0 + 0.08 * (b // 2 - 1))))
        order = np.argsort(-field.reshape(-1), kind="stable")[:min(n, gh * gw)]
        out.append(np.sort(order).astype(np.int32))
    return out


def _normal(seed, stream, shape, std=1.0, dtype=torch.float32):
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 16 + stream)
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dtype)


def _storage(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _valid(case, seed):
    if not case["padded"]:
        return None
    return np.random.default_rng([int(seed), 3]).integers(20, M + 1, case["batch"]).astype(np.int32)


def _deltas(seed, n, most=M):
    return sorted(int(v) for v in np.random.default_rng([int(seed), 4]).choice(most, size=n, replace=False))


def _text(case, seed, token_mode):
    return _normal(seed, 5, (case["batch"], M, C if token_mode else TEXT), dtype=_storage(case))


def _slots(case, seed):
    """One step's cached keys, values and block outputs, [batch, layers, 3, N * C]."""
    n = case["gh"] * case["gw"] * C
    s = torch.empty((case["batch"], case["layers"], 3, n), dtype=_storage(case), device="cuda")
    for i, std in enumerate((2.0, 0.7, 1.5)):
        for b in range(case["batch"]):
            s[b, :, i] = _normal(seed, 6, (case["layers"], n), std) if i == b == 0 else s[0, :, 0].roll(
                977 * (3 * b + i), -1) * (std / 2.0)
    return s


def _step_inputs(case, seed):
    shape = (case["batch"], 4, 2 * case["gh"], 2 * case["gw"]) if case["latent"] else (case["batch"], case["gh"] * case["gw"], C)
    x = _normal(seed, 7, shape, dtype=torch.float32 if case["latent"] else _storage(case))
    traj = _normal(seed, 8, shape) if case["latent"] else None
    if case["guided"]:
        for t in (x, traj):
            t[1::2] = t[0::2]
    t_vec = None if case["latent"] else _normal(seed, 9, (C,))
    return x, traj, t_vec


def _maps(case, seed):
    """Attention sums over heads and blocks: noise, and in every column of a chain an ellipse of high values where the
    edited thing is, at a place drawn for the chain but always the same size and inside the grid with its dilation, so
    that inputs of any seed give lists of the same length."""
    gh, gw = case["gh"], case["gw"]
    rng = np.random.default_rng([int(seed), 10])
    a = rng.uniform(0, 1, (case["batch"], gh, gw, case["n_delta"])).astype(np.float32)
    yy, xx = np.meshgrid(np.arange(gh), np.arange(gw), indexing="ij")
    for b in range(case["batch"]):
        ry, rx = 0.2 * gh, (0.15 + 0.03 * (b % 3)) * gw
        cy = rng.integers(math.ceil(ry) + 2, gh - math.ceil(ry) - 2)
        cx = rng.integers(math.ceil(rx) + 2, gw - math.ceil(rx) - 2)
        a[b][((yy - cy) / ry) ** 2 + ((xx - cx) / rx) ** 2 <= 1.0] += 4.0
    return a.reshape(case["batch"], gh * gw, case["n_delta"])


def _logits(case, seed):
    return _normal(seed, 11, (case["layers"], HEADS, case["gh"] * case["gw"], M), dtype=torch.bfloat16)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "maps":
        return dict(kind=kind, logits=_logits(case, seed), delta=_deltas(seed, case["n_delta"]))
    shape = _shape(case)
    if kind == "localize":
        model = RegionCacheModel(shape, _weights(dict(layers=1), seed, False))
        return dict(kind=kind, model=model, maps=torch.from_numpy(_maps(case, seed)).cuda(), n=case["n_delta"],
                    radius=case["radius"])
    model = RegionCacheModel(shape, _weights(case, seed, shape.token_mode))
    txt = _text(case, seed, shape.token_mode)
    if kind == "text":
        return dict(kind=kind, model=model, txt=txt)
    B = case["batch"]
    s = dict(kind=kind, model=model, tkv=model.prepare_text(txt), case=case)
    s["cache"] = model.alloc_cache(B, 1, host=kind == "hosted")
    n = B * case["layers"] * 3 * case["gh"] * case["gw"] * C
    s["slots"] = s["cache"]._typed(0, n, model.dtype).view(B, case["layers"], 3, -1)
    if kind != "dense":
        s["slots"].copy_(_slots(case, seed))
        s["act"] = ActiveSet.from_lists(_regions(case, seed))
    x, traj, t_vec = _step_inputs(case, seed)
    if case["latent"]:
        for b in range(B):
            s["cache"].latent(b, 1).copy_(traj[b])
    valid = _valid(case, seed)
    s.update(x=x, t_vec=t_vec, out=torch.empty_like(x) if case["latent"] else None,
             valid=None if valid is None else torch.from_numpy(valid).cuda(),
             delta=_deltas(seed, case["n_delta"], 20) if case["n_delta"] else None,
             maps=torch.zeros((B, case["gh"] * case["gw"], case["n_delta"]), device="cuda") if case["n_delta"] else None)
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    kind = s["kind"]
    if kind == "maps":
        return maps_from_logits(s["logits"], s["delta"])
    m = s["model"]
    if kind == "localize":
        mask, act = m.localize(s["maps"], s["n"], 0.3, s["radius"])
        return {"mask": mask, "idx": act.idx[:act.total], "offsets": act.offsets}
    if kind == "text":
        return m.prepare_text(s["txt"]).view(m.dtype)
    if s["maps"] is not None:
        s["maps"].zero_()
    more = dict(delta=s["delta"], maps=s["maps"], latent_out=s["out"], t_vec=s["t_vec"], text_valid=s["valid"],
                guidance=GUIDANCE if s["case"]["guided"] else None)
    if kind == "dense":
        m.build_cache(s["cache"], 0, s["x"], T_NOW, T_NEXT, s["tkv"], **more)
    else:
        m.reuse_step(s["cache"], 0, s["act"], s["x"], T_NOW, T_NEXT, s["tkv"], **more)
    out = {"K": s["slots"][:, :, 0], "V": s["slots"][:, :, 1], "H": s["slots"][:, :, 2]}
    if s["out"] is not None:
        out["latent"] = s["out"]
    if s["maps"] is not None:
        out["maps"] = s["maps"]
    return out


# ------------------------------------------------------------------ what a pass cannot do without

def _rows(case):
    return sum(len(i) for i in _regions(case, 0)) if case["kind"] != "dense" else case["batch"] * case["gh"] * case["gw"]


def work(case):
    kind = case["kind"]
    if kind == "localize":
        n = case["batch"] * case["gh"] * case["gw"]
        return {"bytes": n * (4 * case["n_delta"] + 1), "flops": 0}
    if kind == "maps":
        n = case["layers"] * HEADS * case["gh"] * case["gw"] * M
        return {"bytes": 2 * n, "flops": 4 * n}
    e = 2 if case["dtype"] == "bf16" else 4
    L, B = case["layers"], case["batch"]
    if kind == "text":
        rows = B * M
        return {"bytes": e * (C * TEXT + C * C + L * 2 * C * C + rows * TEXT + L * B * 2 * HEADS * 128 * D),
                "flops": 2 * rows * (C * TEXT + C * C + L * 2 * C * C)}
    N, R = case["gh"] * case["gw"], _rows(case)
    flops = L * R * (2 * (3 * C * C + 3 * C * C + 2 * C * F) + 4 * N * C + 4 * M * C)
    read = L * (6 * C * C + 2 * C * F + B * M * 2 * C) + (0 if kind == "dense" else L * 2 * (B * N - R) * C)
    io = e * (read + L * 3 * R * C) + 4 * B * N * case["n_delta"]
    io += 4 * 16 * B * N * 2 if case["latent"] else e * R * C
    return {"bytes": io, "flops": flops}


def tolerance(case):
    """About four times the measured distance from the same in 64 bits (2-norm), which grows with the blocks and with
    the share of the rows of an output that are computed and not cached."""
    kind = case["kind"]
    if kind == "localize":
        return "exact"  # a mask and whole numbers
    if kind == "maps":
        return {"rel": 1e-6, "max": 4e-5}  # measured 8e-8
    f32 = case["dtype"] == "f32"
    if kind == "text":
        return {"rel": 4e-6} if f32 else {"rel": 1.2e-2}  # bf16: measured 2.9e-3
    if f32:
        return {"rel": 1e-5}  # measured 0.7e-6 to 2.2e-6
    if kind == "dense" or case["layers"] > 5 or case["frac"] > 0.2:
        return {"rel": 3e-2}  # measured 6e-3 to 1e-2, maps 1.5e-2
    return {"rel": 1.3e-2}  # measured 1.2e-3 to 3.8e-3


# ------------------------------------------------------------------ the same in 64 bits

def _f64(a, dtype=None):
    t = torch.as_tensor(np.ascontiguousarray(a)) if isinstance(a, np.ndarray) else a
    t = t.cuda()
    return (t if dtype is None else t.to(dtype)).double()


def _ln(x):
    return torch.nn.functional.layer_norm(x, (x.shape[-1],), eps=1e-6)


def _lin(x, w, b):
    return torch.addmm(b, x, w.t())


def _gelu(x):
    return torch.nn.functional.gelu(x, approximate="tanh")


def _silu(x):
    return x * torch.sigmoid(x)


def _heads(x):
    return x.view(x.shape[0], HEADS, D).transpose(0, 1).contiguous()


def _attend(q, k, v, cols=None):
    """softmax(q k^T / sqrt(72)) v for [heads, n, 72], a head and a few thousand queries at a time; with `cols` also
    the probabilities of those keys, summed over heads."""
    out = torch.empty_like(q)
    maps = torch.zeros((q.shape[1], len(cols)), dtype=q.dtype, device=q.device) if cols else None
    for h in range(HEADS):
        for a in range(0, q.shape[1], 4096):
            p = torch.softmax(q[h, a:a + 4096] @ k[h].t() / math.sqrt(D), -1)
            out[h, a:a + 4096] = p @ v[h]
            if cols:
                maps[a:a + 4096] += p[:, cols]
    return out.transpose(0, 1).reshape(-1, C), maps


def _text64(case, W, txt, dt):
    y = txt.double()
    if "cap_w1" in W:
        y = _lin(_gelu(_lin(y, _f64(W["cap_w1"], dt), _f64(W["cap_b1"]))), _f64(W["cap_w2"], dt), _f64(W["cap_b2"]))
    return y


def _alpha_bar(t):
    return float(np.prod(1.0 - np.linspace(1e-4, 0.02, 1000)[:t + 1]))


def _embed64(case, W, x, dt):
    gh, gw = case["gh"], case["gw"]
    p = x.double().view(4, gh, 2, gw, 2).permute(1, 3, 0, 2, 4).reshape(gh * gw, 16)
    w = 10000.0 ** (-torch.arange(C // 4, dtype=torch.float64, device="cuda") / (C // 4))
    n = torch.arange(gh * gw, device="cuda")
    pos = [f(c.double()[:, None] * w) for c in (n % gw, n // gw) for f in (torch.sin, torch.cos)]
    return _lin(p, _f64(W["pe_w"], dt), _f64(W["pe_b"])) + torch.cat(pos, 1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "localize":
        return None
    if kind == "maps":
        d, z = _deltas(seed, case["n_delta"]), _logits(case, seed)
        return sum(torch.softmax(z[l, h].double(), -1)[:, d] for l in range(case["layers"]) for h in range(HEADS))
    dt = _storage(case)
    token = _shape(case).token_mode
    W = _weights(case, seed, token)
    txt = _text(case, seed, token)
    L, B = case["layers"], case["batch"]
    y = [_text64(case, W, txt[b], dt) for b in range(B)]

    def text_kv(l, b):
        kv = _lin(y[b], _f64(W["layers"][l]["xkv_w"], dt), _f64(W["layers"][l]["xkv_b"]))
        return _heads(kv[:, :C]), _heads(kv[:, C:])

    if kind == "text":
        out = torch.zeros((L, B, 2, HEADS, 128 * D), dtype=torch.float64, device="cuda")
        for l in range(L):
            for b in range(B):
                k, v = text_kv(l, b)
                out[l, b, 0].view(HEADS, 128, D)[:, :M] = k
                out[l, b, 1].view(HEADS, D, 128)[:, :, :M] = v.transpose(1, 2)
        return out.view(-1)

    N = case["gh"] * case["gw"]
    x, traj, t_vec = _step_inputs(case, seed)
    if token:
        temb = t_vec.double()
    else:
        f = 10000.0 ** (-torch.arange(128, dtype=torch.float64, device="cuda") / 128)
        e = torch.cat([torch.cos(T_NOW * f), torch.sin(T_NOW * f)])[None]
        temb = _lin(_silu(_lin(e, _f64(W["temb_w1"], dt), _f64(W["temb_b1"]))), _f64(W["temb_w2"], dt), _f64(W["temb_b2"]))[0]
    t0 = _lin(_silu(temb)[None], _f64(W["tblock_w"], dt), _f64(W["tblock_b"])).view(6, C)
    dense = kind == "dense"
    idx = [torch.arange(N, device="cuda")] * B if dense else [torch.from_numpy(i).long().cuda() for i in _regions(case, seed)]
    slots = torch.zeros((B, L, 3, N * C), dtype=torch.float64, device="cuda") if dense else _slots(case, seed).double()
    valid = _valid(case, seed)
    delta = _deltas(seed, case["n_delta"], 20) if case["n_delta"] else None
    maps = torch.zeros((B, N, case["n_delta"]), dtype=torch.float64, device="cuda") if delta else None
    X = [(x[b].double() if token else _embed64(case, W, x[b], dt))[idx[b]] for b in range(B)]
    for l in range(L):
        w = {k: _f64(v, dt if k in MATS else None) for k, v in W["layers"][l].items()}
        mod = w["sst"] + t0
        for b in range(B):
            K, V = slots[b, l, 0].view(HEADS, N, D), slots[b, l, 1].view(HEADS, N, D)
            qkv = _lin(_ln(X[b]) * (1 + mod[1]) + mod[0], w["qkv_w"], w["qkv_b"])
            K[:, idx[b]], V[:, idx[b]] = _heads(qkv[:, C:2 * C]), _heads(qkv[:, 2 * C:])
            a, _ = _attend(_heads(qkv[:, :C]), K, V)
            X[b] = X[b] + mod[2] * _lin(a, w["proj_w"], w["proj_b"])
            nv = M if valid is None else int(valid[b])
            k, v = text_kv(l, b)
            a, mp = _attend(_heads(_lin(X[b], w["xq_w"], w["xq_b"])), k[:, :nv].contiguous(), v[:, :nv].contiguous(), delta)
            if delta:
                maps[b, idx[b]] += mp
            X[b] = X[b] + _lin(a, w["xproj_w"], w["xproj_b"])
            h = _gelu(_lin(_ln(X[b]) * (1 + mod[4]) + mod[3], w["fc1_w"], w["fc1_b"]))
            X[b] = X[b] + mod[5] * _lin(h, w["fc2_w"], w["fc2_b"])
            slots[b, l, 2].view(N, C)[idx[b]] = X[b]
    out = {"K": slots[:, :, 0], "V": slots[:, :, 1], "H": slots[:, :, 2]}
    if maps is not None:
        out["maps"] = maps
    if not token:
        fs = _f64(W["fin_sst"])
        noise = [_lin(_ln(X[b]) * (1 + fs[1] + temb) + fs[0] + temb, _f64(W["fin_w"], dt), _f64(W["fin_b"])) for b in range(B)]
        if case["guided"]:
            for b in range(0, B, 2):
                noise[b] = noise[b + 1] = noise[b + 1] + GUIDANCE * (noise[b] - noise[b + 1])
        at, an = _alpha_bar(T_NOW), _alpha_bar(T_NEXT)
        ca, cb = math.sqrt(an / at), math.sqrt(1 - an) - math.sqrt(an / at) * math.sqrt(1 - at)
        lat = torch.zeros_like(x, dtype=torch.float64) if dense else traj.double()
        for b in range(B):
            def patches(t):
                return t.view(4, case["gh"], 2, case["gw"], 2).permute(1, 3, 2, 4, 0).reshape(N, 2, 2, 4)
            p = patches(lat[b])
            p[idx[b]] = ca * patches(x[b].double())[idx[b]] + cb * noise[b].view(-1, 2, 2, 8)[..., :4]
            lat[b] = p.view(case["gh"], case["gw"], 2, 2, 4).permute(4, 0, 2, 1, 3).reshape(lat[b].shape)
        out["latent"] = lat
    return out
