"""Timed cases of the verification framework: what a server that uses it has it do.

One round of such a server is: a client's prompt arrives and is prefilled (`ee_prefill`, perhaps
behind rows of image embeddings), then round after round the client's drafted tokens are verified
(`ee_verify` and its batched, sampled and allocation-free forms) and every requested exit's result
leaves early.  The cases time these calls through the package's binding, at the sizes of the
repository's own benchmark and test configurations (4-layer test model, the 1280-wide test model
with a ragged FFN, the Llama2-7B and 13B shapes; the latter two partly cut to fewer layers, which
leaves every layer and head as it is).

Weights are synthetic and the same for every seed: the program has its model loaded.  They are
scaled as in a trained residual network (each layer adds a small part to the stream) and the LM
head is a permutation of the embedding table, so that the model predicts a definite next token
with a probability of about 0.9, as a trained one does, and drafts can follow its continuation
without running it.  Prompts, embedding rows, drafts and the draft model's distributions come from
the seed.  Verify sessions do not commit (`NO_AUTOCOMMIT`): the server repeats a round on the same
state, so every pass of a case has the same context.
"""
import math
import os
import tempfile

import numpy as np
import torch

import eegen
import paper_2505_21594_amd as ee

# name -> (d_model, heads, head_dim, d_ffn, vocab)
SHAPES = {
    "tiny": (256, 4, 64, 688, 1024),
    "mid": (1280, 10, 128, 1072, 3000),
    "7b": (4096, 32, 128, 11008, 32000),
    "13b": (5120, 40, 128, 13824, 32000),
}
ADAPTERS, ADAPTER_WIDTH = 3, 128


def listed():
    return [
        # the repository's smallest configuration: a pass of many very short launches
        dict(name="verify_tiny_g4_ctx64", call="verify", shape="tiny", layers=4, gamma=4, ctx="64", emb=0, exits="2", rows=16),
        # the headline workload: one client, full 7B shape, two exits on the way
        dict(name="verify_7b_g4_ctx512", call="verify", shape="7b", layers=32, gamma=4, ctx="512", emb=0, exits="8,16", rows=16),
        # a long context and more drafts per round
        dict(name="verify_7b_g8_ctx2048", call="verify", shape="7b", layers=32, gamma=8, ctx="2048", emb=0, exits="8,16,24", rows=16),
        # the wider model, an odd number of rows
        dict(name="verify_13b_g5_ctx1024", call="verify", shape="13b", layers=8, gamma=5, ctx="1024", emb=0, exits="4", rows=16),
        # a full tile of 16 rows on an odd context, by a caller that may not allocate
        dict(name="static_7b_g15_ctx129", call="static", shape="7b", layers=8, gamma=15, ctx="129", emb=0, exits="4", rows=16),
        # three clients with contexts of their own in one pass (18 rows)
        dict(name="batch3_7b_g5_ragged", call="batch", shape="7b", layers=8, gamma=5, ctx="700,333,97", emb=0, exits="4", rows=18),
        # eight clients that sent an image (576 embedding rows) and a question, one pass of 40 rows
        dict(name="batch8_7b_g4_vlm", call="batch", shape="7b", layers=8, gamma=4, ctx="64,64,64,64,64,64,64,64", emb=576, exits="4", rows=40),
        # the paper's regime: an exit with adapters after every layer but the last, LM head once per group of exits
        dict(name="exits_7b_g4_adapters", call="adapters", shape="7b", layers=8, gamma=4, ctx="512", emb=0, exits="1,2,3,4,5,6,7", rows=40),
        # probabilistic verification with the draft model's distributions
        dict(name="sampled_7b_g4_ctx512", call="sampled", shape="7b", layers=8, gamma=4, ctx="512", emb=0, exits="2,4", rows=16),
        # a new client's short prompt and its first round, ragged FFN width
        dict(name="prefill_mid_61", call="prefill", shape="mid", layers=3, gamma=4, ctx="61", emb=0, exits="1,2", rows=16),
        # the same for an image prompt on a server that batches
        dict(name="prefill_7b_vlm640", call="prefill", shape="7b", layers=8, gamma=4, ctx="64", emb=576, exits="4", rows=40),
        # the largest: a long prompt on the full model, then its first round
        dict(name="prefill_7b_2041", call="prefill", shape="7b", layers=32, gamma=4, ctx="2041", emb=0, exits="8,16", rows=16),
    ]


def draw(rng):
    def log_size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    call = rng.choice(["verify", "verify", "static", "batch", "batch", "adapters", "sampled", "prefill", "prefill", "prefill"])
    shape = rng.choice(["tiny", "mid", "7b", "7b", "13b"])
    layers = {"tiny": rng.randint(3, 6), "mid": rng.randint(2, 5), "7b": rng.randint(3, 8), "13b": rng.randint(3, 6)}[shape]
    gamma, n, rows, emb = rng.randint(1, 15), 1, 16, 0
    if call == "batch":
        n = rng.randint(2, 12)
        gamma = rng.randint(1, min(15, 48 // n - 1))
        rows = n * (gamma + 1)
    if call == "adapters":
        gamma = rng.randint(1, 9)
        rows = 48 // (gamma + 1) * (gamma + 1)
    if call == "prefill":
        rows = rng.choice([16, 16, 40, 48])
    if call in ("prefill", "batch") and rng.random() < 0.4:
        emb = log_size(16, 576)
    ctx = ",".join(str(log_size(9, 2048 if n == 1 else 800)) for _ in range(n))
    if call == "adapters":
        exits = list(range(1, layers))
    else:
        exits = sorted(rng.sample(range(1, layers), rng.randint(0, min(3, layers - 1))))
    return dict(call=call, shape=shape, layers=layers, gamma=gamma, ctx=ctx, emb=emb, exits=",".join(map(str, exits)), rows=rows)


# ---------------------------------------------------------------- the model

def _config(case):
    d, H, hd, F, V = SHAPES[case["shape"]]
    L = case["layers"]
    n_ad, w = (ADAPTERS, ADAPTER_WIDTH) if case["call"] == "adapters" else (0, 0)
    return eegen.ModelConfig(L, d, H, hd, F, V, tuple(range(1, L)), n_adapters=n_ad, adapter_width=w)


def _generator(name):
    h = 0
    for c in name.encode():
        h = (h * 1000003 + c) % (1 << 61)
    g = torch.Generator(device="cuda")
    g.manual_seed(h)
    return g


def _permutation(V):
    """next_token[t]: the token the model predicts after t."""
    return np.random.default_rng(17).permutation(V)


def _tensor(cfg, name, shape):
    """One weight tensor as bf16 on the GPU, a function of the model's sizes and the tensor's name."""
    d, F, L, V = cfg.d_model, cfg.d_ffn, cfg.n_layers, cfg.vocab
    short = name.split(".")[-1]
    if short == "w_lm":
        # logit of the predicted token about ln(V) + 2, those of the others with the standard deviation s
        s = (math.log(V) + 2.0) / (0.8 * math.sqrt(d))
        inverse = torch.from_numpy(np.argsort(_permutation(V))).cuda()
        return (_tensor(cfg, "emb", (V, d))[inverse].float() * (s / math.sqrt(d))).bfloat16()
    g = _generator("%d.%d.%s" % (d, F, name))
    if short.startswith("g_"):
        return (0.5 + torch.rand(shape, generator=g, device="cuda")).bfloat16()
    residual = 1.0 / math.sqrt(2 * L)
    std = {"emb": 1.0, "wo": residual / math.sqrt(d), "wd": residual / math.sqrt(F)}.get(short)
    if std is None:
        if short.startswith("ad_up"):
            std = 0.3 / math.sqrt(shape[1])
        elif short.startswith("ad_b"):
            std = 0.02
        else:  # projections of a normalised input: outputs with a standard deviation of 1.25
            std = 1.25 / math.sqrt(d)
    return (torch.randn(shape, generator=g, device="cuda") * std).bfloat16()


_models = {}


def _model(case):
    """The loaded model; the server loads it once."""
    cfg = _config(case)
    key = (cfg, case["rows"])
    if key not in _models:
        table, total = eegen.tensor_table(cfg)
        shm = "/dev/shm" if os.access("/dev/shm", os.W_OK) else None
        with tempfile.TemporaryDirectory(dir=shm) as folder:
            path = os.path.join(folder, "model.bin")
            with open(path, "wb") as f:
                f.truncate(total)
                f.write(eegen.format.pack_header(cfg))
                for name, (offset, shape) in table.items():
                    f.seek(offset)
                    f.write(_tensor(cfg, name, shape).view(torch.int16).cpu().numpy().data)
            _models[key] = ee.Model(path, device=0, max_rows=case["rows"])
    return _models[key]


# ---------------------------------------------------------------- inputs

def _inputs(case, seed):
    """Prompts, embedding rows, drafts (and draft distributions) of every session of the case."""
    d, _, _, _, V = SHAPES[case["shape"]]
    follow = _permutation(V)
    sessions = []
    for b, n in enumerate(int(x) for x in case["ctx"].split(",")):
        r = np.random.default_rng([seed, b])
        prompt = r.integers(0, V, n).astype(np.int32)
        emb = None
        if case["emb"]:
            x = torch.from_numpy(r.standard_normal((case["emb"], d), dtype=np.float32))
            emb = x.bfloat16().view(torch.int16).numpy().view(np.uint16)
        pending = int(follow[prompt[-1]])
        greedy, t = [], pending
        for _ in range(case["gamma"]):
            t = int(follow[t])
            greedy.append(t)
        s = dict(prompt=prompt, emb=emb, pending=pending)
        if case["call"] == "sampled":
            s["probs"], s["drafts"], s["u"], s["v"] = eegen.draft_distributions(greedy, V, seed, 0, session=b)
        else:
            p = r.uniform(0.1, 0.6)
            s["drafts"] = np.where(r.random(len(greedy)) < p, r.integers(0, V, len(greedy)), greedy).astype(np.int32)
        sessions.append(s)
    return sorted(sessions, key=lambda s: -len(s["prompt"]))        # the session with the longest context leads a batch


class _State:
    """A server's sessions and the round's inputs; frees the sessions with it."""

    def __init__(self, case, seed):
        self.case = case
        self.exits = [int(x) for x in case["exits"].split(",") if x]
        self.inputs = _inputs(case, seed)
        model = _model(case)
        self.sessions = []
        for b, x in enumerate(self.inputs):
            flags = ee.NO_AUTOCOMMIT | (ee.KEEP_LOGITS if b == 0 else 0) | (ee.SAMPLING if case["call"] == "sampled" else 0)
            n = case["emb"] + len(x["prompt"])
            s = model.session(n + case["gamma"] + 17, max_gamma=case["gamma"], flags=flags)
            self.sessions.append(s)
            if case["call"] != "prefill":
                s.ee_prefill(x["prompt"], emb=x["emb"])
        if case["call"] == "adapters":
            self.sessions[0].ee_session_option(ee.OPT_HEAD_BATCH, 48 // (case["gamma"] + 1))

    def __del__(self):
        for s in self.sessions:
            s.free()


TEMPERATURE = 0.6


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    case, exits = state.case, state.exits
    s, x = state.sessions[0], state.inputs[0]
    out = {}
    if case["call"] == "prefill":
        out["first"] = s.ee_prefill(x["prompt"], emb=x["emb"])
    if case["call"] == "batch":
        ee.ee_verify_batch(state.sessions, [i["drafts"] for i in state.inputs], exits)
    elif case["call"] == "sampled":
        s.ee_verify_sampled(x["drafts"], x["probs"], x["u"], x["v"], TEMPERATURE, exits)
    elif case["call"] == "static":
        s.ee_verify_static(x["drafts"], exits)
    else:
        s.ee_verify(x["drafts"], exits)
    for t in state.sessions:
        t.ee_wait_final()
    results = [t.final_result() for t in state.sessions]
    for name in ("accept_len", "next_token", "final_tokens", "final_conf", "exit_accept_len", "exit_tokens", "exit_conf"):
        out[name] = np.stack([np.asarray(getattr(r, name)) for r in results])
    out["logits"] = s.ee_debug_logits(len(exits))                   # the final head's, of the leading session
    return out


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    d, H, hd, F, V = SHAPES[case["shape"]]
    L, M = case["layers"], case["gamma"] + 1
    A = ADAPTERS * ADAPTER_WIDTH if case["call"] == "adapters" else 0
    heads = len([x for x in case["exits"].split(",") if x]) + 1
    layer = 4 * d * d + 3 * d * F
    bytes_, flops = 2.0 * (L * (layer + 2 * d) + V * d + heads * d + (heads - 1) * 2 * A * d), 0.0
    for n in (int(x) + case["emb"] for x in case["ctx"].split(",")):
        new = M + (n if case["call"] == "prefill" else 0)          # rows that go through the layers
        old = n + M - new                                          # positions cached before the call
        bytes_ += 4.0 * L * d * (old + new) + 2.0 * new * d + 4.0 * M * heads * 2
        flops += 2.0 * L * layer * new + 4.0 * L * d * (new * old + new * (new + 1) / 2)
        flops += 2.0 * M * ((heads * V * d) + (heads - 1) * 2 * A * d)
        if case["call"] == "sampled":
            bytes_ += 4.0 * case["gamma"] * V
        if case["call"] == "prefill":
            flops += 2.0 * V * d
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # Inputs of every product are held to about 17 bits (two bf16 terms): against 64 bits the logits are off by
    # 4e-6 to 5e-6 whatever the shape, two such implementations by up to 1.4 times that; four times as much here.
    return {"rel": 3e-5, "max": 3e-4}


# ---------------------------------------------------------------- the same in 64 bits, plain torch

def exact(case, seed):
    cfg = _config(case)
    d, H, hd, L, eps = cfg.d_model, cfg.n_heads, cfg.head_dim, cfg.n_layers, cfg.rms_eps
    table, _ = eegen.tensor_table(cfg)
    M = case["gamma"] + 1
    exits = [int(x) for x in case["exits"].split(",") if x]
    inputs = _inputs(case, seed)

    def weight(name):
        return _tensor(cfg, name, table[name][1]).double()

    def norm(x, gain):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * gain

    emb = _tensor(cfg, "emb", table["emb"][1])
    streams = []
    for x in inputs:
        tokens = np.concatenate([x["prompt"], [x["pending"]], x["drafts"]]).astype(np.int64)
        h = emb[torch.from_numpy(tokens).cuda()].double()
        if x["emb"] is not None:
            h = torch.cat([torch.from_numpy(x["emb"].view(np.int16)).view(torch.bfloat16).cuda().double(), h])
        streams.append(h)
    del emb
    half = hd // 2
    theta = cfg.rope_base ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / hd)

    def rope(x):                                                    # [rows][H][hd]
        angle = torch.arange(x.shape[0], dtype=torch.float64, device="cuda")[:, None] * theta
        c, s = angle.cos()[:, None], angle.sin()[:, None]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    w_lm = weight("w_lm")
    exit_conf = [[] for _ in inputs]
    for l in range(1, L + 1):
        g_attn, wq, wk, wv, wo = (weight("l%d.%s" % (l, n)) for n in ("g_attn", "wq", "wk", "wv", "wo"))
        for i, h in enumerate(streams):
            x, n = norm(h, g_attn), h.shape[0]
            q, k = (rope((x @ w.t()).view(n, H, hd)) for w in (wq, wk))
            v = (x @ wv.t()).view(n, H, hd)
            o = torch.empty_like(q)
            mask = torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
            for j in range(H):
                score = (q[:, j] @ k[:, j].t()) / math.sqrt(hd)
                o[:, j] = torch.softmax(score.masked_fill(~mask, -math.inf), -1) @ v[:, j]
            streams[i] = h + o.reshape(n, d) @ wo.t()
        del wq, wk, wv, wo
        g_ffn, wg, wu, wd = (weight("l%d.%s" % (l, n)) for n in ("g_ffn", "wg", "wu", "wd"))
        for i, h in enumerate(streams):
            x = norm(h, g_ffn)
            streams[i] = h + (torch.nn.functional.silu(x @ wg.t()) * (x @ wu.t())) @ wd.t()
        del wg, wu, wd
        if l in exits:
            for i, h in enumerate(streams):
                a = h[-M:]
                if cfg.n_adapters:
                    t = torch.nn.functional.silu(a @ weight("ad_down%d" % l).t() + weight("ad_bdown%d" % l))
                    a = a + t @ weight("ad_up%d" % l).t() + weight("ad_bup%d" % l).sum(0)
                z = norm(a, weight("g_exit%d" % l)) @ w_lm.t()
                exit_conf[i].append(torch.softmax(z, -1).amax(-1))
    g_final = weight("g_final")
    z = [norm(h[-M:], g_final) @ w_lm.t() for h in streams]
    out = dict(accept_len=None, next_token=None, final_tokens=None, exit_accept_len=None, exit_tokens=None)
    out["final_conf"] = torch.stack([torch.softmax(t, -1).amax(-1) for t in z])
    out["exit_conf"] = torch.stack([torch.stack(c) if c else torch.empty(0, M, dtype=torch.float64, device="cuda") for c in exit_conf])
    if case["call"] == "prefill":
        out["first"] = None
    out["logits"] = z[0]
    return out
