"""The calls that are timed, and what they have to return.

Every case is one call that a decoding program makes, through the public entry points of the binding: a block-decode
step, a step of the decoded-share stage, a cache refresh (with the length scan that follows it), or the jump controller
between two steps.  The model sizes are the package's own ("8b" and "tiny") and a generic one of 1024 channels; "8b" runs
with its 32 layers in the two steps that a generation spends its time in, and with 8 of them everywhere else.

Weights are the library's seeded normal(0, 0.02) layers.  Embedding and LM head are tied so that the model is as sure of
its next tokens as a trained one: the row of the head that wins at a position is tied to the embedding of the token
held there, by so much that a decoded position's greedy token has a probability between 0 and 1 (which is what a
rounding error moves) and a MASK position's is above the acceptance threshold.  Tokens and masks are drawn from the seed.
"""
import math

import numpy as np
import torch

from paper_2511_21759_amd import binding as B
from paper_2511_21759_amd import workloads as W

WEIGHT_SEED, WEIGHT_STD, TAU = W.WEIGHT_SEED, W.WEIGHT_STD, 0.9
SHAPES = {
    "8b": W.MODEL_SHAPES["8b"],
    "1k": dict(n_layers=8, d_model=1024, n_heads=8, head_dim=128, d_ff=3072, vocab=32000, rope_base=10000.0,
               rms_eps=1e-5, mask_id=31999),
    "tiny": W.MODEL_SHAPES["tiny"],
}
#: deviation of an embedding element, and what the winning logit leads the log-sum of all others by, at decoded and at
#: MASK positions (an estimate: the layers add to it)
EMBED_STD, OVER_DECODED, OVER_MASKED = 8.0, 1.0, 10.0
EOS = 7


def listed():
    return [
        # between two steps: which of eight speculative blocks is adopted, and the next eight (two small launches)
        dict(name="jump-8x32", kind="jump", batch=1, drafts=8, block=32),
        # the smallest model and block: launches and latency only
        dict(name="tiny-step-1x16", kind="step", model="tiny", layers=2, batch=1, prompt=128, resp=64, block=16, drafts=1),
        # a small model's step with the accept-jump drafts: launches, short streams
        dict(name="1k-step-4x32", kind="step", model="1k", layers=8, batch=1, prompt=256, resp=256, block=32, drafts=4),
        # a small model's refresh of three sequences of an odd length
        dict(name="1k-refresh-3x333", kind="refresh", model="1k", layers=8, batch=3, prompt=140, resp=193, scan=False),
        # threshold decoding at full depth: one draft of 32 rows, the weight stream
        dict(name="8b32-step-1x32", kind="step", model="8b", layers=32, batch=1, prompt=256, resp=256, block=32, drafts=1),
        # accept-jump at full depth: block_0 and three speculative blocks, 128 rows
        dict(name="8b32-step-4x32", kind="step", model="8b", layers=32, batch=1, prompt=256, resp=256, block=32, drafts=4),
        # the ragged last block of a response, four drafts of 7 rows behind an odd prompt
        dict(name="8b-step-4x7", kind="step", model="8b", layers=8, batch=1, prompt=301, resp=135, block=7, drafts=4),
        # the decoded-share stage: eight blocks, of which the seven speculative ones hold only what is still masked
        dict(name="8b-shared-8x32", kind="shared", model="8b", layers=8, batch=1, prompt=256, resp=256, block=32, drafts=8),
        # eight plain drafts: 256 rows, between the weight stream and the matrix cores
        dict(name="8b-step-8x32", kind="step", model="8b", layers=8, batch=1, prompt=256, resp=256, block=32, drafts=8),
        # cache refresh behind a few-shot prompt, the longest response that is refreshed there
        dict(name="8b-refresh-1024", kind="refresh", model="8b", layers=8, batch=1, prompt=512, resp=512, scan=False),
        # a refresh of a response that has been cut to an odd length, and the next length scan
        dict(name="8b-refresh-611", kind="refresh", model="8b", layers=8, batch=1, prompt=512, resp=99, scan=True),
        # batched serving: four sequences of 3072 positions, eight drafts of a block of 64 each, 2048 rows
        dict(name="8b-step-4x8x64", kind="step", model="8b", layers=8, batch=4, prompt=2048, resp=1024, block=64, drafts=8),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "shared", "refresh", "refresh", "jump"])
    if kind == "jump":
        return dict(kind="jump", batch=rng.randint(1, 8), drafts=rng.choice([4, 8]), block=rng.randint(5, 64))
    model = rng.choice(["8b", "8b", "8b", "1k", "tiny"])
    layers = 2 if model == "tiny" else 8
    batch = rng.choice([1, 1, 1, 2, 3, 4])
    if kind == "refresh":
        length = _spread(rng, 48, 3072 // batch)
        resp = max(1, int(length * rng.uniform(0.1, 0.7)))
        return dict(kind="refresh", model=model, layers=layers, batch=batch, prompt=length - resp, resp=resp,
                    scan=rng.random() < 0.5)
    drafts = rng.choice([4, 8]) if kind == "shared" else rng.choice([1, 1, 4, 4, 8, rng.randint(2, 7)])
    block = min(_spread(rng, 4, 64), 2048 // (batch * drafts))
    length = _spread(rng, max(64, 2 * block), 3072)
    resp = max(block, int(length * rng.uniform(0.2, 0.6)))
    return dict(kind=kind, model=model, layers=layers, batch=batch, prompt=length - resp, resp=resp, block=block, drafts=drafts)


# ---- inputs -----------------------------------------------------------------------------------------------------

def _shape(case):
    return dict(SHAPES[case["model"]], n_layers=case["layers"])


def _depth_rms(s):
    """Estimated root mean square of what the layers add to an embedding of EMBED_STD (the MLPs do nearly all of it)."""
    gate = WEIGHT_STD * math.sqrt(s["d_model"])
    return math.sqrt(s["n_layers"]) * WEIGHT_STD * math.sqrt(s["d_ff"]) * gate * gate / math.sqrt(2 + 2 * math.pi / (gate * gate + 0.6))


def _tie(s, over):
    """Factor of the tied embedding in a row of the head for a winning logit of log-sum-of-the-others + over."""
    cosine = EMBED_STD / math.hypot(EMBED_STD, _depth_rms(s))
    lse = math.log(s["vocab"]) + 0.5 * WEIGHT_STD ** 2 * s["d_model"]
    return (lse + over) / (cosine * math.sqrt(s["d_model"])) / (EMBED_STD * math.sqrt(s["d_model"]))


def _ends(s):
    """(embedding, LM head) as bf16 on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(WEIGHT_SEED)
    v, d = s["vocab"], s["d_model"]
    embed = torch.empty(v, d, dtype=torch.float32, device="cuda").normal_(0, EMBED_STD, generator=g).bfloat16()
    head = torch.empty(v, d, dtype=torch.float32, device="cuda").normal_(0, WEIGHT_STD, generator=g)
    # token t is followed by t + 1
    head[1:].add_(embed[:-1], alpha=_tie(s, OVER_DECODED))
    head[0].add_(embed[-1], alpha=_tie(s, OVER_MASKED))
    return embed, head.bfloat16()


def _bits(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16).reshape(-1)


_models = {}


def _model(case):
    """The model that a program holds for all its calls."""
    key = (case["model"], case["layers"])
    if key not in _models:
        s = _shape(case)
        m = B.odb_model_create(s)
        B.odb_model_init_random(m, WEIGHT_SEED, WEIGHT_STD)
        embed, head = _ends(s)
        B.odb_model_set_tensor(m, B.T_EMBED, 0, _bits(embed))
        B.odb_model_set_tensor(m, B.T_LM, 0, _bits(head))
        _models[key] = m
    return _models[key]


class _Cache:
    def __init__(self, model, batch, length):
        self.handle = B.odb_cache_create(model, batch, length)

    def __del__(self):
        B.odb_cache_destroy(self.handle)


def _workload(case, seed):
    """Tokens of a half decoded response (three quarters in the decoded-share stage) and the drafts of its first block."""
    p = 0.75 if case["kind"] == "shared" else 0.5
    block = case.get("block", 1)
    return W.decode_workload(_shape(case), case["prompt"], case["resp"], block, case.get("drafts", 1), seed,
                             batch=case["batch"], p_unmasked=p, tau=TAU)


def _jump_inputs(case, seed):
    """Outputs of a step, as the controller meets them: drafts that agree outside their candidates, rising confidences."""
    rng = np.random.default_rng(seed)
    b, S, n = case["block"], case["drafts"], case["batch"]
    mask = SHAPES["8b"]["mask_id"]
    base = np.where(rng.random((n, b)) < 0.5, rng.integers(0, mask, (n, b)), mask).astype(np.int32)
    argmax = np.repeat(rng.integers(0, mask, (n, 1, b)), S, axis=1).astype(np.int32)
    conf = (rng.random((n, S, b)) ** 0.5).astype(np.float32)
    drafts = np.repeat(base[:, None], S, axis=1)
    pos, tok = np.full((n, 4), -1, np.int32), np.zeros((n, 4), np.int32)
    sets = [(), (0,), (1,), (0, 1), (2,), (0, 1, 2), (3,), (0, 1, 2, 3)][:S]
    for i in range(n):
        where = rng.permutation(np.flatnonzero(base[i] == mask))[:4]
        pos[i, :len(where)] = where
        tok[i, :len(where)] = np.where(rng.random(len(where)) < 0.8, argmax[i, 0, where], 3)
        for s, chosen in enumerate(sets):
            for c in chosen:
                if c < len(where):
                    drafts[i, s, where[c]] = tok[i, c]
    unmask = ((drafts == mask) & (conf > 0.6)).astype(np.uint8)
    return drafts, conf, argmax, unmask, pos, tok


def prepare(case, seed):
    if case["kind"] == "jump":
        return dict(case=case, model=_jump_model(), given=[torch.from_numpy(x).cuda() for x in _jump_inputs(case, seed)])
    model, wl = _model(case), _workload(case, seed)
    cache = _Cache(model, case["batch"], wl.tokens.shape[1])
    tokens = torch.from_numpy(wl.tokens).cuda()
    st = dict(case=case, model=model, cache=cache, tokens=tokens)
    if case["kind"] == "refresh":
        return st
    B.odb_prefill(model, cache.handle, tokens, wl.resp_off)
    st["drafts"] = torch.from_numpy(wl.drafts).cuda()
    st["block_off"] = wl.block_off
    st["n_masked"] = int((wl.drafts[:, 0] == _shape(case)["mask_id"]).sum(axis=1).max())
    return st


def _jump_model():
    """The controller takes the MASK id from a model; its other sizes do not matter there."""
    if "jump" not in _models:
        _models["jump"] = B.odb_model_create(dict(SHAPES["tiny"], vocab=SHAPES["8b"]["vocab"], mask_id=SHAPES["8b"]["mask_id"]))
    return _models["jump"]


def run(state):
    case = state["case"]
    if case["kind"] == "jump":
        return B.odb_speculative_jump(state["model"], *state["given"], n_next=case["drafts"])
    if case["kind"] == "refresh":
        conf, argmax = B.odb_prefill(state["model"], state["cache"].handle, state["tokens"], case["prompt"])
        if not case["scan"]:
            return conf, argmax
        return conf, argmax, B.odb_predict_length(state["model"], state["tokens"], conf, argmax, case["prompt"], EOS, TAU)
    if case["kind"] == "shared":
        return B.odb_block_step_shared(state["model"], state["cache"].handle, state["drafts"], state["block_off"], state["n_masked"], TAU)
    return B.odb_block_step(state["model"], state["cache"].handle, state["drafts"], state["block_off"], TAU)


# ---- what a pass cannot do without --------------------------------------------------------------------------------

def work(case):
    if case["kind"] == "jump":
        n, S, b = case["batch"], case["drafts"], case["block"]
        return {"bytes": n * (S * b * (4 + 4 + 4 + 1) + 32 + S * b * 4 + 36), "flops": 0}
    s = _shape(case)
    d, f, v, nl, n = s["d_model"], s["d_ff"], s["vocab"], s["n_layers"], case["batch"]
    length = case["prompt"] + case["resp"]
    weights = 2 * (nl * (4 * d * d + 3 * d * f) + v * d)
    if case["kind"] == "refresh":
        rows, out, keys, moved = n * length, n * case["resp"], length, n * length
    else:
        per = case["drafts"] * case["block"]
        if case["kind"] == "shared":       # a quarter of the block is masked
            per = case["block"] + (case["drafts"] - 1) * math.ceil(case["block"] / 4)
        rows, out, keys, moved = n * per, n * per, length, n * (length - case["block"])
    kv = moved * nl * 2 * d * 2            # read by a step, written by a refresh
    flops = 2.0 * rows * nl * (4 * d * d + 3 * d * f) + 2.0 * out * v * d + 4.0 * rows * keys * d * nl
    return {"bytes": weights + kv + rows * (d * 2 + 4) + out * 9, "flops": flops}


def tolerance(case):
    if case["kind"] == "jump":
        return "exact"
    # Confidences from binary16 operands and 32-bit sums.  Two orders of summation differ by 1.3e-4 after 8 layers and
    # 1.7e-4 to 3.1e-4 after 32, and from 64 bits by as much; four times that.  Whole numbers are decided far from ties: the
    # winning logit leads by several units, and no decision changed between those orders.
    return {"rel": 1.3e-3 if case["layers"] == 32 else 6e-4, "differ": 0.005}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

def _i64(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


_GAMMA, _M1, _M2 = 0x9E3779B97F4A7C15, 0xBF58476D1CE4E5B9, 0x94D049BB133111EB


def _mix(z):
    """SplitMix64's output function (Steele, Lea, Flood 2014) on int64 tensors, whose products wrap."""
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * _i64(_M1)
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * _i64(_M2)
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _first(x):
    return int(_mix(torch.tensor([_i64(x + _GAMMA)]))[0])


def _weight(tensor, layer, rows, cols):
    """One tensor of odb_model_init_random as its header describes it, [rows, cols] float64."""
    key = _first(_first(WEIGHT_SEED) + (tensor << 32 | layer))
    out = torch.empty(rows * cols, dtype=torch.float64, device="cuda")
    for lo in range(0, rows * cols, 1 << 25):
        hi = min(rows * cols, lo + (1 << 25))
        z = _mix(torch.arange(lo + 1, hi + 1, device="cuda") * _i64(_GAMMA) + _i64(key))
        u1 = (((z >> 32) & 0xFFFFFFFF).double() + 0.5) / 2.0 ** 32
        u2 = ((z & 0xFFFFFFFF).double() + 0.5) / 2.0 ** 32
        x = torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * u2)
        out[lo:hi] = (WEIGHT_STD * x).float().bfloat16().double()
    return out.view(rows, cols)


def _norm(s, h):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + s["rms_eps"])


def _rope(s, x, pos):
    half = s["head_dim"] // 2
    freq = s["rope_base"] ** (-torch.arange(half, device="cuda", dtype=torch.float64) / half)
    ang = pos.double()[:, None, None] * freq
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _attend(q, k, v, seen):
    """q [n, H, dh], k, v [m, H, dh], seen [n, m] or None -> [n, H * dh]."""
    out = torch.empty_like(q)
    for h in range(q.shape[1]):
        z = q[:, h].contiguous() @ k[:, h].t().contiguous() / math.sqrt(q.shape[2])
        if seen is not None:
            z = z.masked_fill(~seen, float("-inf"))
        out[:, h] = torch.softmax(z, -1) @ v[:, h].contiguous()
    return out.reshape(q.shape[0], -1)


def _rows_of(case, s, drafts, block_off, length):
    """Rows that a step computes for one sequence: tokens, positions, which keys each sees (the cached ones, then the
    rows themselves), and where each row's result goes in [S, b]."""
    S, b = drafts.shape
    dev = dict(device="cuda")
    if case["kind"] == "step":
        where = torch.arange(S * b, **dev)
    else:
        masked = torch.nonzero(drafts[0] == s["mask_id"]).flatten()
        where = torch.cat([torch.arange(b, **dev)] + [k * b + masked for k in range(1, S)])
    draft, at = where // b, where % b
    own = draft[:, None] == draft[None, :]
    if case["kind"] == "shared":           # block_0's decoded positions are seen by all
        decoded = (drafts[0] != s["mask_id"])[at] & (draft == 0)
        own = own | decoded[None, :]
    outside = torch.ones(length, dtype=torch.bool, **dev)
    outside[block_off:block_off + b] = False
    seen = torch.cat([outside.expand(len(where), length), own], 1)
    return drafts.reshape(-1)[where], block_off + at, seen, where


def exact(case, seed):
    if case["kind"] == "jump":
        return None
    s, wl = _shape(case), _workload(case, seed)
    d, f, H, dh, length = s["d_model"], s["d_ff"], s["n_heads"], s["head_dim"], case["prompt"] + case["resp"]
    embed, head = _ends(s)
    step = case["kind"] != "refresh"
    ctx_tokens = torch.from_numpy(wl.tokens).cuda().long()
    ctx_pos = torch.arange(length, device="cuda")
    ctx = embed[ctx_tokens].double()                                 # [batch, length, d]
    rows, new = [], []
    if step:
        for i in range(case["batch"]):
            rows.append(_rows_of(case, s, torch.from_numpy(wl.drafts[i]).cuda().long(), wl.block_off, length))
            new.append(embed[rows[i][0]].double())
    for layer in range(s["n_layers"]):
        wq, wk, wv, wo = (_weight(t, layer, d, d).t() for t in (B.T_WQ, B.T_WK, B.T_WV, B.T_WO))
        wg, wu = (_weight(t, layer, f, d).t() for t in (B.T_WG, B.T_WU))
        wd = _weight(B.T_WD, layer, d, f).t()
        for i in range(case["batch"]):
            def attention(h, pos, more, seen):
                x = _norm(s, h)
                q, k, v = (x @ w for w in (wq, wk, wv))
                q, k, v = _rope(s, q.view(-1, H, dh), pos), _rope(s, k.view(-1, H, dh), pos), v.view(-1, H, dh)
                keys, values = (k, v) if more is None else (torch.cat([more[0], k]), torch.cat([more[1], v]))
                h = h + _attend(q, keys, values, seen) @ wo
                x = _norm(s, h)
                return h + (torch.nn.functional.silu(x @ wg) * (x @ wu)) @ wd, (k, v)
            ctx[i], kv = attention(ctx[i], ctx_pos, None, None)
            if step:
                new[i], _ = attention(new[i], rows[i][1], kv, rows[i][2])
    del embed
    conf = torch.zeros(wl.drafts.shape if step else (case["batch"], case["resp"]), dtype=torch.float64, device="cuda")
    for i in range(case["batch"]):
        x = _norm(s, new[i] if step else ctx[i, case["prompt"]:])
        z = torch.cat([x @ part.double().t() for part in head.split(16384)], 1)
        p = torch.exp(z.max(-1).values - torch.logsumexp(z, -1))
        if step:
            conf[i].view(-1)[rows[i][3]] = p
        else:
            conf[i] = p
    none = (None, None) if step or case["scan"] else (None,)
    return (conf,) + none
