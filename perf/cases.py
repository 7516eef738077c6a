"""Performance cases: the calls a decode is made of, at the sizes it meets.

A user of this package builds a Model over bf16 (or, for the tiny
configuration, float32) weights, usually packs them, and decodes: every
denoising step is one full forward (embedding, layers, head on the block rows)
or, with key/value reuse, a forward of the block rows against the cache.  The
cases are those pieces through the package's public calls: single layers and
pairs of layers at each workload's sequence shape, the block rows of a cached
step, the LM head, and short whole forwards that return logits.

Model widths are the package's own configurations (LLaDA-8B, Dream-7B and the
tiny float32 model).  A layer's time does not depend on how many layers follow
it, so cases run one to four of them; cases without a head use a small
vocabulary, which only the embedding gather sees.
"""
import math

import torch

from paper_2608_22646_amd import binding, synth

CONFIGS = {"llada": synth.LLADA_8B, "dream": synth.DREAM_7B, "tiny": synth.TINY}
SMALL_VOCAB = 4096


def _case(kind, model, layers, B, P, G, rows, packed, name=None):
    c = {"kind": kind, "model": model, "layers": layers, "B": B, "P": P, "G": G, "rows": rows, "packed": packed}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one denoising step (forward, head, commit, flag) of the tiny model; launches and latency
        _case("step", "tiny", 2, 1, 32, 64, 32, False, "step_tiny"),
        # the float32 path at a ragged length and a small batch, logits wanted
        _case("forward", "tiny", 2, 4, 141, 96, 32, False, "forward_tiny_b4"),
        # the headline decode's layers: LLaDA-8B widths, batch 1, 256 + 256 tokens
        _case("layer", "llada", 2, 1, 256, 256, 32, True, "layer_llada_b1"),
        # batch 8, 512 + 512 tokens: the large GEMMs
        _case("layer", "llada", 1, 8, 512, 512, 32, True, "layer_llada_b8"),
        # Dream-7B widths (grouped heads, 37888 gate/up columns), 512 + 256 tokens
        _case("layer", "dream", 2, 1, 512, 256, 32, True, "layer_dream_b1"),
        # a long-context prompt: attention weighs most here
        _case("layer", "dream", 1, 1, 8192, 256, 32, True, "layer_dream_long"),
        # prompts are rarely a multiple of eight: three sequences of 365 tokens, weights not packed (the default)
        _case("layer", "llada", 1, 3, 301, 64, 32, False, "layer_llada_ragged"),
        # a whole forward with its logits: layers with the folded residual sums, final norm, LM head on one block
        _case("forward", "llada", 2, 1, 256, 256, 32, True, "forward_llada_b1"),
        # a cached step's forward, batch 1: 32 block rows stream every weight once
        _case("block_forward", "llada", 2, 1, 256, 256, 32, True, "block_llada_b1"),
        # the cached step's layers at batch 8: 256 block rows
        _case("block_layer", "llada", 2, 8, 512, 512, 32, True, "block_llada_b8"),
        # the cached step's layers behind a long prompt of odd length
        _case("block_layer", "dream", 2, 1, 8001, 256, 32, True, "block_dream_long"),
        # LM head and vocabulary reduction of a batch-8 step
        _case("head", "llada", 0, 8, 512, 512, 32, True, "head_llada_b8"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "block_layer", "block_layer", "forward", "block_forward", "head", "step"])
    rows = rng.choice([16, 32, 32, 32, 64])
    if kind == "step":
        G = rows * rng.randint(1, 4)
        return _case("step", "tiny", 2, rng.randint(1, 4), _log(rng, 8, 256), G, rows, False)
    model = "tiny" if kind == "forward" and rng.random() < 0.25 else rng.choice(["llada", "llada", "dream"])
    B = min(rng.choice([1, 1, 1, 2, 3, 4, 5, 8]), 256 // rows)
    top = 512 if model == "tiny" else 8192
    G = rows * max(1, min(512, _log(rng, 32, 512)) // rows)
    P = _log(rng, 16, max(32, top // B - G))
    if rng.random() < 0.35:  # a third of the prompts at a multiple of eight
        P = max(8, P // 8 * 8)
    layers = 2 if model == "tiny" or kind in ("forward", "block_forward") else 0 if kind == "head" else (
        1 if kind == "layer" and B * (P + G) > 2048 else 2)
    if kind == "forward" and model != "tiny":
        layers = 1 if B * (P + G) > 2048 else 2
    packed = model != "tiny" and rng.random() < 0.75
    return _case(kind, model, layers, B, P, G, rows, packed)


# ---------------------------------------------------------------- inputs
def _config(c):
    cfg = CONFIGS[c["model"]]
    kw = {"n_layers": c["layers"]}
    if c["kind"] in ("layer", "block_layer"):
        kw["vocab"] = SMALL_VOCAB
    return synth.reduced(cfg, **kw)


def _generator(seed, i):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * (seed + 1) + i)
    return g


def _weights(cfg, seed):
    out = []
    for i, (_, shape, std) in enumerate(synth.weight_specs(cfg)):
        g = _generator(seed, i)
        if std is None:  # norm gains around 1
            w = 1.0 + 0.1 * torch.randn(shape, generator=g, device="cuda")
        else:
            w = torch.randn(shape, generator=g, device="cuda").mul_(std)
        out.append(w.to(cfg.torch_dtype))
    return out


def _tokens(cfg, c, seed):
    """[B, L] token ids of a decode in its first block: a prompt, then masks."""
    x = torch.randint(0, cfg.vocab - 1, (c["B"], c["P"] + c["G"]), generator=_generator(seed, 900), device="cuda",
                      dtype=torch.int32)
    x[:, c["P"]:] = cfg.vocab - 1
    if c["kind"].startswith("block"):  # some of the block is committed since the last refresh
        x[:, c["P"]:c["P"] + c["rows"]:2] = torch.randint(0, cfg.vocab - 1, (c["B"], (c["rows"] + 1) // 2), device="cuda",
                                                         generator=_generator(seed, 901), dtype=torch.int32)
    return x


def _cache_views(cfg, kv, B, L):
    """[(K [B, Hkv, L, hd], V^T [B, Hkv, hd, L])] per layer of a bf16 model's cache buffer."""
    n = B * cfg.n_kv_heads * L * cfg.head_dim
    slab = (2 * n + 255) // 256 * 256
    out = []
    for l in range(cfg.n_layers):
        k = kv[2 * l * slab:2 * l * slab + 2 * n].view(torch.bfloat16).view(B, cfg.n_kv_heads, L, cfg.head_dim)
        v = kv[(2 * l + 1) * slab:(2 * l + 1) * slab + 2 * n].view(torch.float16)
        out.append((k, v.view(B, cfg.n_kv_heads, cfg.head_dim, L)))
    return out


def _fill_cache(cfg, views, seed):
    """Keys and values as a refresh stores them: bf16 values of projections of normed rows."""
    std = 0.02 * math.sqrt(cfg.d_model)
    for l, (k, v) in enumerate(views):
        k.copy_(torch.randn(k.shape, generator=_generator(seed, 920 + 2 * l), device="cuda").mul_(std))
        t = torch.randn(v.shape, generator=_generator(seed, 921 + 2 * l), device="cuda").mul_(std)
        v.copy_(t.to(torch.bfloat16))


def _hidden(cfg, c, seed):
    """A final residual [B*L, d]: its rows' scale varies, as it does in a model."""
    M = c["B"] * (c["P"] + c["G"])
    h = torch.randn((M, cfg.d_model), generator=_generator(seed, 940), device="cuda")
    return h.mul_(torch.rand((M, 1), generator=_generator(seed, 941), device="cuda").mul_(3.0).add_(0.5))


def prepare(case, seed):
    c = case
    cfg = _config(c)
    B, L = c["B"], c["P"] + c["G"]
    model = binding.Model(cfg, _weights(cfg, seed))
    if c["packed"]:
        model.pack_weights()
    s = {"c": c, "cfg": cfg, "model": model, "B": B, "L": L, "ws": model.workspace(B, L, c["rows"])}
    lay = model.layout(B, L, c["rows"])
    kind = c["kind"]
    if kind == "step":
        s["prompt"] = _tokens(cfg, c, seed)[:, :c["P"]].contiguous()
        s["st"] = binding.DecodeState(B, c["P"], c["G"])
        s["ctl"] = binding.Controller(block_len=c["rows"])
    elif kind == "head":
        h = s["ws"][lay.h:lay.h + B * L * cfg.d_model * 4].view(torch.float32).view(B * L, cfg.d_model)
        h.copy_(_hidden(cfg, c, seed))
    else:
        s["x"] = _tokens(cfg, c, seed)
    n = B * (c["rows"] if kind == "block_layer" else L)
    if kind in ("layer", "block_layer"):
        s["h"] = s["ws"][lay.h:lay.h + n * cfg.d_model * 4].view(torch.float32).view(n, cfg.d_model)
    if kind.startswith("block"):
        s["kv"] = model.kv_cache(B, L)
        s["kv"].zero_()
        s["views"] = _cache_views(cfg, s["kv"], B, L)
        _fill_cache(cfg, s["views"], seed)
    torch.cuda.synchronize()
    return s


# ---------------------------------------------------------------- one pass
def run(state):
    s, c, m = state, state["c"], state["model"]
    kind, B, L, P, rows = c["kind"], s["B"], s["L"], c["P"], c["rows"]
    if kind == "step":
        st = s["st"]
        m.state_init(s["prompt"], c["G"], st)
        done, conf, arg = m.step(s["ctl"], st, 0, 0, s["ws"], record=True)
        return {"conf": conf, "argmax": arg, "x": st.x, "commit_step": st.commit_step, "reason": st.reason, "s": st.s,
                "budget": st.budget, "ell": st.ell, "done": st.done, "all_done": done}
    if kind == "forward":
        conf, _, logits = m.forward(s["x"], P, rows, ws=s["ws"], logits=True)
        return {"conf": conf, "logits": logits}
    if kind == "layer":
        m.embed(s["x"], s["ws"])
        for l in range(c["layers"]):
            m.layer(l, 2, B, L, s["ws"])
        return {"h": s["h"]}
    if kind == "block_forward":
        conf, _, logits = m.forward_kv(s["x"], P, rows, s["kv"], False, ws=s["ws"], logits=True)
        return {"conf": conf, "logits": logits, "kv": s["views"]}
    if kind == "block_layer":
        m.embed_rows(s["x"], P, rows, s["ws"])
        for l in range(c["layers"]):
            m.layer_kv(l, 2, B, L, P, rows, s["kv"], s["ws"])
        return {"h": s["h"], "kv": s["views"]}
    conf, arg, _ = m.head(B, L, P, rows, s["ws"])
    return {"conf": conf, "argmax": arg}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    c, cfg = case, _config(case)
    B, L, rows = c["B"], c["P"] + c["G"], c["rows"]
    size = 4 if cfg.dtype == "f32" else 2
    block = c["kind"].startswith("block")
    M = B * (rows if block else L)
    d, F, V = cfg.d_model, cfg.d_ff, cfg.vocab
    per_layer = d * (cfg.q_dim + 2 * cfg.kv_dim) + cfg.q_dim * d + 3 * d * F
    flops = c["layers"] * (2 * M * per_layer + 4 * M * L * cfg.q_dim)
    nbytes = c["layers"] * (per_layer + 2 * d) * size
    if c["kind"] != "head":  # token ids and the embedding rows in
        nbytes += M * 4 + M * d * size
    if c["kind"] in ("layer", "block_layer"):
        nbytes += M * d * 4
    else:  # the head's rows, its weights, and what it writes
        R = B * rows
        flops += 2 * R * V * d
        nbytes += V * d * size + d * size + R * 8
        if c["kind"] == "head":
            nbytes += R * d * 4
        if c["kind"] in ("forward", "block_forward"):
            nbytes += R * V * 4
    if block:  # the other positions' keys and values in, the block's out
        nbytes += c["layers"] * 2 * B * L * cfg.kv_dim * size
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    kind = case["kind"]
    if case["model"] == "tiny":  # float32, sums in float64
        return {"rel": 1e-5}
    # Two correct bf16 implementations round some operands to neighbouring bf16
    # values.  Against 64 bits without any rounding: layers 0.55-0.85% (1.5% for
    # 80 cached rows), the head's confidences 0.12-0.42%, logits of two layers
    # about 0.5% and their confidences about 2%.
    if kind == "head":  # an argmax moves only at a tie of the logits
        return {"rel": 1e-2, "differ": 0.01}
    return {"rel": 0.03, "max": 0.9} if kind in ("forward", "block_forward") else {"rel": 0.02, "max": 0.8}


# ---------------------------------------------------------------- the same in 64 bits
def _norm(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _rope(x, pos, base):
    """Rotate-half RoPE of [..., n, hd] at positions pos [n]."""
    half = x.shape[-1] // 2
    ang = pos[:, None] * base ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / x.shape[-1])[None]
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _mm(a, w):
    return a @ w.double().T


def _layer64(cfg, w, h, B, n, pos, cache=None):
    """One layer on h [B*n, d] at positions pos; cache: float64 (K, V^T) of every position, updated in place."""
    hd, eps = cfg.head_dim, cfg.rms_eps
    a = _norm(h, w[0].double(), eps)
    heads = lambda t, H: t.view(B, n, H, hd).transpose(1, 2)  # noqa: E731
    q = _rope(heads(_mm(a, w[1]), cfg.n_heads), pos, cfg.rope_base)
    k = _rope(heads(_mm(a, w[2]), cfg.n_kv_heads), pos, cfg.rope_base)
    v = heads(_mm(a, w[3]), cfg.n_kv_heads)
    if cache is not None:
        p0 = int(pos[0])
        cache[0][:, :, p0:p0 + n] = k
        cache[1][:, :, :, p0:p0 + n] = v.transpose(2, 3)
        k, v = cache[0], cache[1].transpose(2, 3)
    o = torch.empty((B, n, cfg.n_heads, hd), dtype=torch.float64, device=h.device)
    rep = cfg.n_heads // cfg.n_kv_heads
    for b in range(B):
        for j in range(cfg.n_heads):
            sc = q[b, j] @ k[b, j // rep].T.contiguous() / math.sqrt(hd)
            o[b, :, j] = torch.softmax(sc, -1) @ v[b, j // rep].contiguous()
            del sc
    h = h + _mm(o.reshape(B * n, -1), w[4])
    a = _norm(h, w[5].double(), eps)
    u = torch.nn.functional.silu(_mm(a, w[6])) * _mm(a, w[7])
    return h + _mm(u, w[8])


def _head64(cfg, w, h):
    """(logits, confidences, argmax) of rows h."""
    lg = _mm(_norm(h, w[-2].double(), cfg.rms_eps), w[-1])
    masked = lg.clone()
    masked[:, cfg.vocab - 1] = -math.inf
    p = torch.softmax(masked, -1)
    return lg, p.max(-1).values, p.argmax(-1)


def exact(case, seed):
    c = case
    cfg = _config(c)
    B, L, P, rows = c["B"], c["P"] + c["G"], c["P"], c["rows"]
    w = _weights(cfg, seed)
    kind = c["kind"]
    block = kind.startswith("block")
    if kind == "head":
        h = _hidden(cfg, c, seed).double().view(B, L, -1)[:, P:P + rows].reshape(B * rows, -1)
        _, conf, arg = _head64(cfg, w, h)
        return {"conf": conf.view(B, rows), "argmax": None}
    x = _tokens(cfg, c, seed)
    n, p0 = (rows, P) if block else (L, 0)
    h = w[0][x[:, p0:p0 + n].reshape(-1).long()].double()
    pos = torch.arange(p0, p0 + n, device="cuda", dtype=torch.float64)
    kv = None
    if block:
        size = cfg.n_layers * 2 * ((2 * B * cfg.n_kv_heads * L * cfg.head_dim + 255) // 256 * 256)
        views = _cache_views(cfg, torch.zeros(size, dtype=torch.uint8, device="cuda"), B, L)
        _fill_cache(cfg, views, seed)
        kv = [(k.double(), v.double()) for k, v in views]
    for l in range(c["layers"]):
        h = _layer64(cfg, w[1 + 9 * l:10 + 9 * l], h, B, n, pos, kv[l] if block else None)
    if kind == "layer":
        return {"h": h}
    if kind == "block_layer":
        return {"h": h, "kv": kv}
    lg, conf, _ = _head64(cfg, w, h if block else h.view(B, L, -1)[:, P:P + rows].reshape(B * rows, -1))
    if kind == "step":  # the decisions are whole numbers; s holds the block's first-step confidences
        s = torch.zeros((B, c["G"]), dtype=torch.float64, device="cuda")
        s[:, :rows] = conf.view(B, rows)
        return {"conf": conf.view(B, rows), "argmax": None, "x": None, "commit_step": None, "reason": None, "s": s,
                "budget": None, "ell": None, "done": None, "all_done": None}
    out = {"conf": conf.view(B, rows), "logits": lg.view(B, rows, -1)}
    if block:
        out["kv"] = kv
    return out
