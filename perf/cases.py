"""What the shard forward is measured on: the calls that a program which serves a Ladder-Residual model makes.

Every case takes the library through its Python binding, as bench.py and the tests do.  The shapes are the ones the
framework is configured for (`paper_2501_06589_amd.inputs.WORKLOADS`): the 1.2B and 8B models whole on one GPU, one
rank's shard of the 70B shape at R = 8 and R = 4, and the tiny fp32 model with both of its shards computed.  A case
holds a few layers of the stack (the layers are alike; enough of them that a decode step's weights do not fit the
last-level cache), so that what is compared is the layer and not the growth of a rounding through eighty of them.

Kinds:
  decode    a cache handed over by another process (ladder_load_kv), then `steps` decode steps
  prefill   one prefill call
  generate  a prefill, then `steps` decode steps on the cache that it left
  stage     the same, as one stage of a pipeline (three tensors in, three out)
  head      token embedding, and final norm + output projection + greedy token, for one position per sequence
"""
import math

import torch

from paper_2501_06589_amd import ladder

# per-shard sizes: hidden, query heads, kv heads, head size, SwiGLU size, R, computed shards, rotary base
MODELS = {
    "tiny": dict(dtype="fp32", hidden=256, nq=2, nkv=1, d=64, inter=344, tp=2, shards=2, theta=1e4),
    "1.2b": dict(dtype="bf16", hidden=2048, nq=16, nkv=8, d=128, inter=5632, tp=1, shards=1, theta=1e4),
    "8b": dict(dtype="bf16", hidden=4096, nq=32, nkv=8, d=128, inter=14336, tp=1, shards=1, theta=5e5),
    "70b_r8": dict(dtype="bf16", hidden=8192, nq=8, nkv=1, d=128, inter=3584, tp=8, shards=1, theta=5e5),
    "70b_r4": dict(dtype="bf16", hidden=8192, nq=16, nkv=2, d=128, inter=7168, tp=4, shards=1, theta=5e5),
}
GROWTH = 128      # cache capacity beyond the prompt: the 128 generated tokens of the configurations
EPS = 1e-5
DEV = "cuda:0"


def _case(kind, model, **kw):
    c = dict(kind=kind, model=model, layers=1, batch=1, prompt=0, cached=0, steps=0, wiring="ladder", standard_layers=0,
             graph=False, vocab=0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest calls: the fp32 model of the parity runs, prompt and answer; launches and latency count
        _case("generate", "tiny", name="tiny_fp32_generate", layers=2, prompt=32, steps=8),
        # the headline: token-by-token generation of a 70B rank at R = 8, batch 4, behind a prompt of 1024 tokens
        _case("decode", "70b_r8", name="decode_70b_r8_b4", layers=8, batch=4, cached=1024, steps=8),
        # one user of an 8B model
        _case("decode", "8b", name="decode_8b_b1", layers=4, batch=1, cached=2048, steps=8),
        # a small model that serves a batch: short layers
        _case("decode", "1.2b", name="decode_1.2b_b16", layers=12, batch=16, cached=1024, steps=8),
        # the largest batch of the paper's throughput sweep (1, 4, 16, 64)
        _case("decode", "8b", name="decode_8b_b64", layers=2, batch=64, cached=1024, steps=8),
        # long conversations: 32 k cached positions, ragged against every tile
        _case("decode", "70b_r8", name="decode_70b_r8_32k", layers=4, batch=4, cached=32001, steps=8),
        # the prefill-heavy configuration: 16 prompts of 2048 tokens at once, one layer
        _case("prefill", "70b_r4", name="prefill_70b_r4_16x2048", layers=1, batch=16, prompt=2048),
        # time to first token of one ordinary prompt
        _case("prefill", "8b", name="prefill_8b_1x2048", layers=2, batch=1, prompt=2048),
        # a chat turn: a prompt that fills no tile
        _case("prefill", "8b", name="prefill_8b_1x100", layers=4, batch=1, prompt=100),
        # a few ragged prompts and the first tokens of their answers
        _case("generate", "1.2b", name="generate_1.2b_3x333", layers=8, batch=3, prompt=333, steps=8),
        # one stage of a pipeline, a long prompt of odd length and the first tokens behind it
        _case("stage", "70b_r8", name="stage_70b_r8_1x4001", layers=2, batch=1, prompt=4001, steps=4),
        # what stands around the stack in every step of generation: embedding, logits and greedy tokens, batch 16
        _case("head", "8b", name="head_8b_b16", batch=16, vocab=128256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _params(m):
    return m["hidden"] * (2 * m["nq"] + 2 * m["nkv"]) * m["d"] + 3 * m["hidden"] * m["inter"]


def _rows_most(m):
    """Rows of a prefill that cost one layer of the model what the largest listed case costs."""
    r4 = MODELS["70b_r4"]
    return 16 * 2048 * _params(r4) // (_params(m) * m["shards"])


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["prefill"] * 3 + ["generate"] * 2 + ["stage", "head"])
    model = rng.choice(["70b_r8", "70b_r4"] if kind == "stage" else ["1.2b", "8b", "70b_r8"] if kind == "head" else
                       ["1.2b", "8b", "70b_r8", "70b_r4"] if rng.random() < 0.85 else ["tiny"])
    m = MODELS[model]
    if kind == "head":
        return _case("head", model, batch=_log_int(rng, 1, 64), vocab=rng.choice([16032, 32000, 128256]))
    layers = 2 if model == "tiny" else rng.choice([2, 3, 4])
    if kind == "decode":
        batch = _log_int(rng, 1, 4 if model == "tiny" else 64)
        cached = _log_int(rng, 17, 600) if model == "tiny" else min(_log_int(rng, 64, 32768), 64 * 8 * 1024 // (batch * m["nkv"]))
        wiring = "ladder" if kind == "stage" or rng.random() < 0.6 else rng.choice(["standard", "parallel", "hybrid"])
        return _case("decode", model, layers=layers, batch=batch, cached=cached, steps=rng.choice([4, 6, 8]),
                     wiring="ladder" if wiring == "hybrid" else wiring, standard_layers=1 if wiring == "hybrid" else 0,
                     graph=rng.random() < 0.2)
    batch = _log_int(rng, 1, 2 if model == "tiny" else 16)
    prompt = _log_int(rng, 3, 300) if model == "tiny" else _log_int(rng, 16, 8192)
    layers = 2 if model == "tiny" else rng.choice([1, 2])
    while batch > 1 and batch * prompt * layers > _rows_most(m):
        batch //= 2
    layers = layers if batch * prompt * layers <= _rows_most(m) else 1
    return _case(kind, model, layers=layers, batch=batch, prompt=prompt, steps=0 if kind == "prefill" else rng.choice([4, 6, 8]))


def _inputs(case, seed):
    """Weights, peers, cache and stream of the case, from the seed alone."""
    m = MODELS[case["model"]]
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    dt = torch.float32 if m["dtype"] == "fp32" else torch.bfloat16

    def normal(*shape, std=1.0, mean=0.0, dtype=dt):
        return torch.randn(shape, generator=g, device=DEV).mul_(std).add_(mean).to(dtype)

    H, I, d, nq, nkv, B = m["hidden"], m["inter"], m["d"], m["nq"], m["nkv"], case["batch"]
    z = dict(m=m, dt=dt)
    if case["kind"] == "head":
        z["table"], z["final_norm"] = normal(case["vocab"], H), normal(H, std=0.02, mean=1.0)
        z["w_lm"] = normal(H, case["vocab"], std=0.02)
        z["tokens"] = torch.randint(0, case["vocab"], (B,), generator=g, device=DEV, dtype=torch.int32)
        z["x"] = normal(B, H, std=2.0, dtype=torch.float32)
        return z
    z["layers"] = []
    for _ in range(case["layers"]):
        an, mn = normal(H, std=0.02, mean=1.0), normal(H, std=0.02, mean=1.0)
        z["layers"].append([dict(attn_norm=an, mlp_norm=mn, wq=normal(H, nq * d, std=0.02), wk=normal(H, nkv * d, std=0.02),
                                 wv=normal(H, nkv * d, std=0.02), wo=normal(nq * d, H, std=0.02), w_gate=normal(H, I, std=0.02),
                                 w_up=normal(H, I, std=0.02), w_down=normal(I, H, std=0.02)) for _ in range(m["shards"])])
    peers = m["tp"] - m["shards"]
    z["peers"] = normal(2, peers, B * max(case["prompt"], 1), H, std=0.02) if peers else None
    if case["cached"]:
        z["kv"] = [[(normal(B, nkv, case["cached"], d), normal(B, nkv, case["cached"], d)) for _ in range(m["shards"])]
                   for _ in range(case["layers"])]
    if case["kind"] == "stage":     # the stream as an earlier stage leaves it, fp32
        z["hand"] = [normal(B, case["prompt"], H, std=s, dtype=torch.float32) for s in (1.0, 0.3, 0.3)]
        z["hands"] = [[normal(B, H, std=s, dtype=torch.float32) for s in (1.0, 0.3, 0.3)] for _ in range(case["steps"])]
    else:
        z["x"] = normal(B, case["prompt"], H) if case["prompt"] else None
        z["xs"] = [normal(B, H) for _ in range(case["steps"])]
    return z


def prepare(case, seed):
    """A context with the layers loaded, and the inputs in device memory."""
    z = _inputs(case, seed)
    m, B = z["m"], case["batch"]
    prompt = max(case["prompt"], 1)
    wiring = dict(ladder=ladder.LADDER_WIRING_LADDER, standard=ladder.LADDER_WIRING_STANDARD, parallel=ladder.LADDER_WIRING_PARALLEL)
    cfg = ladder.make_config(
        n_layers=case["layers"], hidden=m["hidden"], n_q_heads=m["nq"], n_kv_heads=m["nkv"], head_dim=m["d"], inter=m["inter"],
        tp_degree=m["tp"], n_real_shards=m["shards"], max_batch=B, max_seq=max(case["prompt"], case["cached"]) + GROWTH,
        max_tokens=prompt, dtype=ladder.LADDER_FP32 if m["dtype"] == "fp32" else ladder.LADDER_BF16, wiring=wiring[case["wiring"]],
        n_standard_layers=case["standard_layers"], decode_graph=1 if case["graph"] else 0, rms_eps=EPS, rope_theta=m["theta"],
        peer_pool=2 if m["tp"] > m["shards"] else 0, peer_rows=B * prompt if m["tp"] > m["shards"] else 0)
    ctx = ladder.Ladder(cfg)
    if case["kind"] == "head":
        ctx.load_head(z["table"], z["final_norm"], z["w_lm"])
        del z["table"], z["w_lm"]
    else:
        for i, shards in enumerate(z["layers"]):
            for r, w in enumerate(shards):
                ctx.load_layer(i, r, w)
        torch.cuda.synchronize()     # the weights are copied: a program drops its own
        del z["layers"]
        if z["peers"] is not None:
            ctx.set_peer_partials(z["peers"])
    z["ctx"], z["kind"] = ctx, case["kind"]
    return z


def run(state):
    ctx, kind = state["ctx"], state["kind"]
    if kind == "head":
        emb = ctx.embed(state["tokens"])
        logits, tokens = ctx.head(state["x"])
        return dict(emb=emb, logits=logits, tokens=tokens)
    if kind == "stage":
        out = dict(prompt=ctx.prefill_stage(state["hand"]))
        out["steps"] = [ctx.decode_step_stage(h) for h in state["hands"]]
        return out
    out = {}
    if kind == "decode":
        for i, shards in enumerate(state["kv"]):
            for r, (k, v) in enumerate(shards):
                ctx.load_kv(i, r, k, v)
    else:
        out["prompt"] = ctx.prefill(state["x"])
    out["steps"] = [ctx.decode_step(x) for x in state["xs"]]
    return out


def work(case):
    m, B, L, T, S = MODELS[case["model"]], case["batch"], case["layers"], case["prompt"], case["cached"]
    e = 4 if m["dtype"] == "fp32" else 2
    H = m["hidden"]
    if case["kind"] == "head":
        return {"bytes": H * case["vocab"] * e + B * (2 * H * e + 4 * H + 4 * case["vocab"] + 8), "flops": 2.0 * B * H * case["vocab"]}
    weights = L * m["shards"] * _params(m)
    kv_row = L * m["shards"] * m["nkv"] * m["d"] * 2 * e              # one position of one sequence
    head_flops = 4.0 * L * m["shards"] * m["nq"] * m["d"]             # one query against one position
    peers = 2 * L * (m["tp"] - m["shards"]) * H * e                   # of one row
    io = 3 * 8 * H if case["kind"] == "stage" else (4 + e) * H        # stream in and out of one row
    by, fl = 0.0, 0.0
    if case["kind"] == "decode":
        by += 2.0 * B * S * kv_row                                    # the cache that is handed over: read and written
    else:
        rows = B * T
        by += weights * e + rows * (peers + io + kv_row)
        fl += 2.0 * weights * rows + head_flops * B * T * (T + 1) / 2
    for i in range(case["steps"]):
        n = max(T, S) + i + 1
        by += weights * e + B * (n * kv_row + peers + io)
        fl += 2.0 * weights * B + head_flops * B * n
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # about four times the error that was measured against 64 bits
    if MODELS[case["model"]]["dtype"] == "fp32":
        return {"rel": 1e-6, "max": 1e-5}                     # 32-bit sums in another order
    if case["kind"] == "head":
        return {"rel": 7e-3, "max": 5e-2, "differ": 0.01}     # the normed rows are rounded to bf16 once
    if case["kind"] == "decode" and case["batch"] <= 16:
        return {"rel": 2e-4, "max": 4e-3}                     # 16 significant bits between modules; a cache entry may round the other way
    if case["kind"] == "stage":
        return {"rel": 3e-2, "max": 0.5}                      # one attention output by itself: the small mean over thousands of positions
    return {"rel": 2e-2, "max": 0.15}                         # bf16 operands between the modules


# -- the same in 64 bits ----------------------------------------------------------------------------------------

def _norm(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _rope(x, pos, theta):        # x [B, T, heads, d], adjacent pairs
    d = x.shape[-1]
    ang = torch.arange(pos, pos + x.shape[1], device=x.device, dtype=torch.float64)[:, None] * \
        theta ** (-torch.arange(0, d, 2, device=x.device, dtype=torch.float64) / d)
    c, s = torch.cos(ang)[None, :, None, :], torch.sin(ang)[None, :, None, :]
    a, b = x[..., 0::2], x[..., 1::2]
    return torch.stack([a * c - b * s, a * s + b * c], -1).flatten(-2)


def _attention(y, w, z, cache, pos):
    m, dt = z["m"], z["dt"]
    B, T, _ = y.shape
    d, nq, nkv = m["d"], m["nq"], m["nkv"]
    heads = lambda p, n: (y @ w[p].double()).view(B, T, n, d)     # noqa: E731
    q, k, v = _rope(heads("wq", nq), pos, m["theta"]), _rope(heads("wk", nkv), pos, m["theta"]), heads("wv", nkv)
    k, v = (t.transpose(1, 2).to(dt) for t in (k, v))              # the cache holds the storage type
    if cache.get("k") is not None and pos:
        k, v = torch.cat([cache["k"], k], 2), torch.cat([cache["v"], v], 2)
    cache["k"], cache["v"] = k, v
    S, out = pos + T, torch.empty(B, T, nq, d, device=y.device, dtype=torch.float64)
    hide = torch.arange(S, device=y.device)[None, :] > torch.arange(pos, S, device=y.device)[:, None]
    for b in range(B):
        for h in range(nq):
            kh, vh = k[b, h // (nq // nkv)].double(), v[b, h // (nq // nkv)].double()
            p = (q[b, :, h] @ kh.t() / math.sqrt(d)).masked_fill_(hide, -math.inf)
            out[b, :, h] = torch.softmax(p, -1) @ vh
    return out.view(B, T, nq * d) @ w["wo"].double()


def _mlp(y, w):
    g = y @ w["w_gate"].double()
    return (g * torch.sigmoid(g) * (y @ w["w_up"].double())) @ w["w_down"].double()


def _forward(case, z, caches, streams, pos):
    """streams: {0: x_0, -1: x_{-1}} [B, T, H]; returns the list x_0 .. x_2N and the module outputs."""
    L = case["layers"]
    x, hs = dict(streams), {}
    B, T, H = x[0].shape
    for mod in range(1, 2 * L + 1):
        layer = (mod - 1) // 2
        lag = 1 if case["wiring"] == "standard" or layer < case["standard_layers"] else 2
        if case["wiring"] == "parallel":
            lag = 1 if mod % 2 else 2
        src = x.get(mod - lag, x[0])
        h = 0.0
        for r, w in enumerate(z["layers"][layer]):
            if mod % 2:
                h = h + _attention(_norm(src, w["attn_norm"]), w, z, caches[layer][r], pos)
            else:
                h = h + _mlp(_norm(src, w["mlp_norm"]), w)
        if z["peers"] is not None:
            h = h + z["peers"][mod % 2][:, :B * T].double().sum(0).view(B, T, H)
        hs[mod], x[mod] = h, x[mod - 1] + h
    return x, hs


def exact(case, seed):
    z = _inputs(case, seed)
    if case["kind"] == "head":
        y = _norm(z["x"].double(), z["final_norm"])
        logits = torch.cat([y @ w.double() for w in z["w_lm"].split(8192, 1)], 1)
        return dict(emb=z["table"][z["tokens"].long()].double(), logits=logits, tokens=None)
    L, R, n = case["layers"], z["m"]["shards"], 2 * case["layers"]
    caches = [[dict(k=z["kv"][i][r][0], v=z["kv"][i][r][1]) if case["kind"] == "decode" else {} for r in range(R)] for i in range(L)]
    pos = case["cached"]

    def call(x, T):      # x: the embeddings, or a stage's three tensors
        nonlocal pos
        if case["kind"] == "stage":
            res, att, mlp = (t.double().view(case["batch"], T, -1) for t in x)
            xs, hs = _forward(case, z, caches, {-1: res + att, 0: res + att + mlp}, pos)
            got = (xs[n - 2], hs[n - 1], hs[n])
        else:
            xs, _ = _forward(case, z, caches, {0: x.double().view(case["batch"], T, -1)}, pos)
            got = (xs[n],)
        pos += T
        return got if case["kind"] == "stage" else got[0]

    def step(x):
        got = call(x, 1)
        return tuple(t[:, 0] for t in got) if case["kind"] == "stage" else got[:, 0]

    out = {}
    if case["prompt"]:
        out["prompt"] = call(z["hand"] if case["kind"] == "stage" else z["x"], case["prompt"])
    out["steps"] = [step(x) for x in (z["hands"] if case["kind"] == "stage" else z["xs"])]
    return out
