"""The calls whose speed counts: denoising steps and LM-head calls as a serving
program makes them through ``paper_2606_29094_amd.engine`` and ``.dlm``.

A step case is one ``Engine`` step of a model with the layer shapes of the
repository's configurations (MHA-8B, GQA-7B, the tiny fp32 model) and their
full vocabularies; the bf16 models keep 2 to 4 layers, each of full width,
since every layer of the deep models is the same work. A head case is one
``dlm.head_confidence`` call. Requests of one case differ in prompt length and
active block; which lengths they have follows from the case alone ("mix"), the
weights, tokens and mask positions follow from the seed.
"""
import math
import random

import numpy as np
import torch

from paper_2606_29094_amd import dlm, engine

# layer shapes and calibrated 1/tau of the repository's three models
MODELS = {
    "tiny-fp32": dict(d=256, hq=4, hkv=4, dh=64, ffn=688, vocab=2048, dtype="f32", inv_tau=13.1),
    "mha-8b": dict(d=4096, hq=32, hkv=32, dh=128, ffn=12288, vocab=126464, dtype="bf16",
                   inv_tau=8.018),
    "gqa-7b": dict(d=3584, hq=28, hkv=4, dh=128, ffn=18944, vocab=152064, dtype="bf16",
                   inv_tau=11.626),
}
EPS, THETA, THRESHOLD = 1e-5, 10000.0, 0.9
MAX_ROWS = 65536           # recomputed rows of the largest step


def _step(name, model, layers, mode, batch, prompt, gen, block, refresh=0, stats=False, masked=0.7,
          mix=0):
    """prompt: (shortest, longest); refresh: requests that recompute their
    whole sequence in the step (the others make a cache step)."""
    return {"name": name, "kind": "step", "model": model, "layers": layers, "mode": mode,
            "batch": batch, "prompt_lo": prompt[0], "prompt_hi": prompt[1], "gen": gen,
            "block": block, "refresh": refresh, "stats": stats, "masked": masked, "mix": mix}


def listed():
    return [
        # the whole fp32 model, one request, no cache: the smallest call, all latency
        _step("tiny-exact-b1", "tiny-fp32", 2, "none", 1, (64, 64), 64, 32, refresh=1,
              masked=1.0),
        # LM head of one request's block: the vocabulary matrix streamed once
        {"name": "head-mha-32", "kind": "head", "model": "mha-8b", "rows": 32},
        # one user decoding with a dual cache: 32 rows per step, weights streamed
        _step("mha-decode-b1", "mha-8b", 4, "dual", 1, (261, 261), 256, 32, masked=1.0),
        # three users of the GQA model, blocks of 64, the last one ragged
        _step("gqa-decode-b3", "gqa-7b", 4, "dual", 3, (90, 700), 200, 64, mix=3),
        # the repository's batch of 8, dual cache: 256 rows over 1280 positions
        _step("mha-dual-b8", "mha-8b", 4, "dual", 8, (1024, 1024), 256, 32),
        # one request without a cache: 512 rows, each step exact
        _step("mha-exact-b1", "mha-8b", 4, "none", 1, (256, 256), 256, 32, refresh=1,
              masked=1.0),
        # batch of 8, prefix cache: block and everything after it, ragged rows
        _step("mha-prefix-b8", "mha-8b", 2, "prefix", 8, (1024, 1024), 256, 32, mix=1),
        # continuous batching: 32 requests of mixed lengths, two of them entering a
        # new block, confidence statistics on
        _step("mha-mixed-b32", "mha-8b", 2, "dual", 32, (128, 2048), 256, 32, refresh=2, stats=True,
              mix=5),
        # prefill / first step of a block for a batch of 8
        _step("mha-refresh-b8", "mha-8b", 2, "dual", 8, (1024, 1024), 256, 32, refresh=8,
              masked=1.0),
        # the default benchmark's batch of 64: a pure cache step of 4096 rows
        _step("gqa-dual-b64", "gqa-7b", 2, "dual", 64, (512, 512), 512, 64, masked=0.4, mix=2),
        # the same batch with three requests entering a new block
        _step("gqa-mixed-b64", "gqa-7b", 2, "dual", 64, (512, 512), 512, 64, refresh=3, masked=0.4,
              mix=2),
        # the same batch, every request recomputed: 65536 rows, the largest call
        _step("gqa-refresh-b64", "gqa-7b", 2, "dual", 64, (512, 512), 512, 64, refresh=64,
              masked=1.0),
    ]


def draw(rng):
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    what = rng.random()
    if what < 0.15:
        return {"kind": "head", "model": rng.choice(["mha-8b", "gqa-7b"]), "rows": log(1, 4096)}
    if what < 0.25:
        c = _step("", "tiny-fp32", 2, rng.choice(["none", "dual", "prefix"]), log(1, 12),
                  (1, log(1, 200)), log(8, 128), rng.choice([8, 16, 32, 48]))
    else:
        model = rng.choice(["mha-8b", "gqa-7b"])
        lo = log(16, 1024)
        c = _step("", model, 2, rng.choice(["none", "dual", "dual", "prefix"]), log(1, 64),
                  (lo, min(2048, int(lo * rng.uniform(1, 4)))), rng.choice([128, 200, 256, 512]),
                  rng.choice([32, 32, 64, 64, 24, 57]))
    c["mix"] = rng.randrange(1 << 20)
    c["stats"] = rng.random() < 0.25
    c["masked"] = rng.choice([1.0, 0.7, 0.4, 0.2]) if c["batch"] >= 8 else 1.0
    if c["mode"] == "none" or rng.random() < 0.2:
        c["refresh"] = c["batch"]
    elif rng.random() < 0.5:
        c["refresh"] = rng.randint(1, max(1, c["batch"] // 8))
    while sum(r1 - r0 for r0, r1 in _rows(c)) > MAX_ROWS // 4:
        c["batch"] = (c["batch"] + 1) // 2
        c["refresh"] = min(c["refresh"], c["batch"])
    del c["name"]
    return c


# ------------------------------------------------------------------ shapes
def _shapes(case):
    """(prompt length, active block index, masked positions of the block) of each request."""
    r = random.Random(case["mix"])
    out = []
    nblk = -(-case["gen"] // case["block"])
    for _ in range(case["batch"]):
        p = r.randint(case["prompt_lo"], case["prompt_hi"])
        k = r.randrange(nblk)
        n = min(case["block"], case["gen"] - k * case["block"])
        out.append((p, k, max(1, round(case["masked"] * n))))
    return out


def _rows(case):
    """Recomputed positions [r0, r1) of each request; the first ``refresh``
    requests recompute their whole sequence."""
    out = []
    for i, (p, k, _) in enumerate(_shapes(case)):
        s, end = p + k * case["block"], p + case["gen"]
        if i < case["refresh"] or case["mode"] == "none":
            out.append((0, end))
        elif case["mode"] == "dual":
            out.append((s, min(s + case["block"], end)))
        else:
            out.append((s, end))
    return out


def _weights(m, layers, seed, head_only=False):
    """Random-init weights in the library's layouts: N(0, 0.02), gains near 1."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.bfloat16 if m["dtype"] == "bf16" else torch.float32
    mat = lambda r, c: torch.empty(r, c, dtype=dt, device="cuda").normal_(0, 0.02, generator=gen)
    gain = lambda: torch.empty(m["d"], device="cuda").normal_(1.0, 0.05, generator=gen)
    qd = m["hq"] * m["dh"]
    t = {"lm_head": mat(m["vocab"], m["d"]), "final_norm": gain()}
    t["embed"] = t["lm_head"] if head_only else mat(m["vocab"], m["d"])
    t["layers"] = [{"attn_norm": gain(), "w_qkv": mat(qd + 2 * m["hkv"] * m["dh"], m["d"]),
                    "w_o": mat(m["d"], qd), "ffn_norm": gain(),
                    "w_gate_up": mat(2 * m["ffn"], m["d"]), "w_down": mat(m["d"], m["ffn"])}
                   for _ in range(layers)]
    return t


def _tokens(case, seed):
    """Per request (tokens, mask, confidences of the unmasked output tokens)."""
    rng = np.random.default_rng(seed)
    vocab = MODELS[case["model"]]["vocab"]
    out = []
    for p, k, masked in _shapes(case):
        end, s = p + case["gen"], p + k * case["block"]
        n = min(case["block"], end - s)
        tok = rng.integers(0, vocab - 1, end).astype(np.int32)
        mask = np.zeros(end, np.uint8)
        mask[s + n:] = 1
        mask[s + rng.permutation(n)[:masked]] = 1
        tok[mask != 0] = vocab - 1
        conf = np.where(mask[p:] != 0, 0, rng.uniform(0.3, 1.0, case["gen"])).astype(np.float32)
        out.append((tok, mask, np.concatenate([np.zeros(p, np.float32), conf])))
    return out


def _model(m, layers, t):
    shape = engine.ModelShape(layers, m["d"], m["hq"], m["hkv"], m["dh"], m["ffn"], m["vocab"],
                              m["dtype"], EPS, THETA, m["vocab"] - 1)
    return engine.DeviceModel(shape, t, m["inv_tau"])


def _head_rows(case, seed):
    m = MODELS[case["model"]]
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    return torch.empty(case["rows"], m["d"], dtype=torch.bfloat16,
                       device="cuda").normal_(0, 1, generator=g)


# ------------------------------------------------------------------- cases
def prepare(case, seed):
    m = MODELS[case["model"]]
    if case["kind"] == "head":
        # a model handle whose one layer is never run
        small = dict(m, ffn=64)
        model = _model(small, 1, _weights(small, 1, seed, head_only=True))
        n = case["rows"]
        ws = torch.empty(dlm.workspace_bytes(model.handle, n, min(64, -(-n // 64))),
                         dtype=torch.uint8, device="cuda")
        return {"case": case, "model": model, "u": _head_rows(case, seed), "ws": ws,
                "conf": torch.zeros(n, device="cuda"),
                "tok": torch.zeros(n, dtype=torch.int32, device="cuda")}
    model = _model(m, case["layers"], _weights(m, case["layers"], seed))
    shapes, rows = _shapes(case), _rows(case)
    longest = max(p for p, _, _ in shapes) + case["gen"]
    eng = engine.Engine(model, case["batch"], longest, case["mode"],
                        max_rows=max(sum(r1 - r0 for r0, r1 in rows), longest),
                        stats=case["stats"])
    eng.cache_buf.zero_()
    reqs = []
    for (p, k, _), (tok, mask, conf) in zip(shapes, _tokens(case, seed)):
        r = engine.Request(tok[:p], case["gen"], case["block"], THRESHOLD)
        eng.admit(r, m["vocab"] - 1)
        eng.set_state(r, tok, mask, k, conf if case["stats"] else None)
        reqs.append(r)
    if case["mode"] != "none":
        for r in reqs[case["refresh"]:]:      # the block's recompute step lies behind these
            eng.refresh([r])
    torch.cuda.synchronize()
    return {"case": case, "eng": eng, "reqs": reqs, "tokens": eng.tokens.clone(),
            "mask": eng.mask.clone(),
            "tok_conf": eng.tok_conf.clone() if case["stats"] else None}


def run(state):
    if "u" in state:
        dlm.head_confidence(state["model"].handle, state["u"], state["case"]["rows"],
                            state["conf"], state["tok"], state["ws"])
        return {"conf": state["conf"], "tok": state["tok"]}
    eng, reqs = state["eng"], state["reqs"]
    # the tokens and masks of the batch as the scheduler holds them
    eng.tokens.copy_(state["tokens"])
    eng.mask.copy_(state["mask"])
    if state["tok_conf"] is not None:
        eng.tok_conf.copy_(state["tok_conf"])
    for r in reqs[:state["case"]["refresh"]]:
        r.refreshed_block = -1               # these enter a new block
    eng.enqueue_step(reqs)
    n = len(reqs)
    out = {"conf": eng.block_conf[:n * dlm.DLM_MAX_BLOCK].view(n, dlm.DLM_MAX_BLOCK),
           "kv": eng.cache_buf.view(eng.model.shape.torch_dtype), "tokens": eng.tokens,
           "mask": eng.mask}
    if state["tok_conf"] is not None:
        out["stats"] = eng.stats[:n * dlm.DLM_NSTATS].view(n, dlm.DLM_NSTATS)
    return out


def work(case):
    m = MODELS[case["model"]]
    es = 2 if m["dtype"] == "bf16" else 4
    d, v = m["d"], m["vocab"]
    if case["kind"] == "head":
        n = case["rows"]
        return {"bytes": es * (v * d + n * d) + 8 * n, "flops": 2 * n * d * v}
    shapes, rows = _shapes(case), _rows(case)
    n = sum(r1 - r0 for r0, r1 in rows)
    lens = [p + case["gen"] for p, _, _ in shapes]
    masked = sum(x for _, _, x in shapes)
    par = d * (m["hq"] + 2 * m["hkv"]) * m["dh"] + m["hq"] * m["dh"] * d + 3 * d * m["ffn"]
    kv = 2 * m["hkv"] * m["dh"] * es                    # one position's keys and values
    attn = sum(4 * (r1 - r0) * length * m["hq"] * m["dh"] for (r0, r1), length in zip(rows, lens))
    stale = sum(length - (r1 - r0) for (r0, r1), length in zip(rows, lens))
    return {"bytes": case["layers"] * (es * par + kv * (stale + n)) + es * (v * d + n * d),
            "flops": case["layers"] * (2 * n * par + attn) + 2 * masked * d * v}


def tolerance(case):
    # fp32: sums in another order (6e-6 against 64 bits for the head, 1e-6 for
    # the fp32 model). A bf16 step: one-ulp changes of stored bf16 values, which
    # 1/tau of about 10 turns into 0.2-1.5 % of the confidences when every
    # projection's sums are split differently (0.5-2.8 % against 64 bits).
    # Tokens and masks: a confidence that crosses the threshold, 0.2 % seen.
    if case["kind"] == "head":
        return {"rel": 5e-5, "max": 5e-4, "differ": 0.002}
    if case["model"] == "tiny-fp32":
        return {"rel": 1e-5, "max": 5e-4, "differ": 0.01}
    return {"rel": 0.03, "max": 0.4, "differ": 0.01}


# ------------------------------------------------- the same in 64-bit torch
def _norm(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g.double()


def _rope(x, pos):
    half = x.shape[-1] // 2
    freq = THETA ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    a = (pos.double()[:, None] * freq)[:, None, :]
    c, s = torch.cos(a), torch.sin(a)
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _forward(m, t, toks, slots, rows, kv):
    """Layers over the rows of each request; kv: per layer (K [slot, head, pos,
    dh], V [slot, head, dh, pos]), updated. Returns the rows' final values."""
    hq, hkv, dh = m["hq"], m["hkv"], m["dh"]
    hs = [t["embed"][tok[r0:r1].long()].double() for tok, (r0, r1) in zip(toks, rows)]
    pos = [torch.arange(r0, r1, device="cuda") for r0, r1 in rows]
    for layer, (K, V) in zip(t["layers"], kv):
        w = {k: v.double() for k, v in layer.items()}
        for i, (h, ps, slot) in enumerate(zip(hs, pos, slots)):
            length = toks[i].numel()
            x = _norm(h, w["attn_norm"]) @ w["w_qkv"].T
            q = _rope(x[:, :hq * dh].view(-1, hq, dh), ps)
            K[slot][:, ps] = _rope(x[:, hq * dh:(hq + hkv) * dh].view(-1, hkv, dh), ps).transpose(0, 1)
            V[slot][:, :, ps] = x[:, (hq + hkv) * dh:].view(-1, hkv, dh).permute(1, 2, 0)
            o = torch.empty_like(q)
            for j in range(hkv):
                gq = q[:, j * (hq // hkv):(j + 1) * (hq // hkv)]
                p = torch.softmax(gq.reshape(-1, dh) @ K[slot, j, :length].T.contiguous() / math.sqrt(dh), -1)
                o[:, j * (hq // hkv):(j + 1) * (hq // hkv)] = (
                    p @ V[slot, j, :, :length].T.contiguous()).view(-1, hq // hkv, dh)
            h = h + o.reshape(-1, hq * dh) @ w["w_o"].T
            y = _norm(h, w["ffn_norm"]) @ w["w_gate_up"].T
            g = y[:, :m["ffn"]]
            h = h + (g * torch.sigmoid(g) * y[:, m["ffn"]:]) @ w["w_down"].T
            hs[i] = h
        del w
    return hs


def _confidence(m, lm_head, u):
    """max softmax of the scaled logits of the rows u."""
    mx = torch.full((u.shape[0],), -math.inf, dtype=torch.float64, device="cuda")
    s = torch.zeros_like(mx)
    for c in range(0, m["vocab"], 16384):
        z = (u @ lm_head[c:c + 16384].double().T) * m["inv_tau"]
        new = torch.maximum(mx, z.amax(-1))
        s = s * torch.exp(mx - new) + torch.exp(z - new[:, None]).sum(-1)
        mx = new
    return 1.0 / s


def exact(case, seed):
    m = MODELS[case["model"]]
    if case["kind"] == "head":
        small = dict(m, ffn=64)
        t = _weights(small, 1, seed, head_only=True)
        u = _head_rows(case, seed).double()
        conf = torch.cat([_confidence(m, t["lm_head"], x) for x in u.split(4096)])
        return {"conf": conf, "tok": None}
    t = _weights(m, case["layers"], seed)
    shapes, rows, toks = _shapes(case), _rows(case), _tokens(case, seed)
    dev = [torch.from_numpy(tok).cuda() for tok, _, _ in toks]
    longest = max(p for p, _, _ in shapes) + case["gen"]
    s_max, b = (longest + 63) // 64 * 64, case["batch"]
    buf = torch.zeros(2 * case["layers"], b, m["hkv"] * s_max * m["dh"], dtype=torch.float64,
                      device="cuda")
    kv = [(buf[2 * i].view(b, m["hkv"], s_max, m["dh"]),
           buf[2 * i + 1].view(b, m["hkv"], m["dh"], s_max)) for i in range(case["layers"])]
    # the engine hands out slots 0, 1, ... in the order of admission
    slots = list(range(b))
    if case["mode"] != "none" and case["refresh"] < b:
        f = case["refresh"]
        _forward(m, t, dev[f:], slots[f:], [(0, x.numel()) for x in dev[f:]], kv)
    hs = _forward(m, t, dev, slots, rows, kv)
    conf = torch.full((b, dlm.DLM_MAX_BLOCK), -1.0, dtype=torch.float64, device="cuda")
    where, us = [], []
    for i, ((p, k, _), (r0, _), (_, mask, _)) in enumerate(zip(shapes, rows, toks)):
        s = p + k * case["block"]
        n = min(case["block"], p + case["gen"] - s)
        at = np.nonzero(mask[s:s + n])[0]
        where += [(i, int(a)) for a in at]
        us.append(_norm(hs[i][torch.from_numpy(at + s - r0).cuda()], t["final_norm"]))
    c = _confidence(m, t["lm_head"], torch.cat(us))
    at = torch.tensor(where, device="cuda")
    conf[at[:, 0], at[:, 1]] = c
    out = {"conf": conf, "kv": buf.view(-1), "tokens": None, "mask": None}
    if case["stats"]:
        out["stats"] = None
    return out
