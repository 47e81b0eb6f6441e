"""GPU checks of the bf16 attention kernels at the edges of their dispatch and of
their tiles, on exactly the values each launch received (dlm_debug_trace),
against fp64 softmax attention over the slot's cached keys and values. The cache
holds NaN wherever no step wrote, so a read past a sequence that reaches the
result shows."""
import numpy as np
import pytest
import torch

from kernel_checks import U, half_ulp
from paper_2606_29094_amd import dlm, engine

pytestmark = pytest.mark.gpu


def _model(gpu, hq, hkv, dh, seed, ffn=64):
    d, V = 128, 65
    g = torch.Generator().manual_seed(seed)
    mat = lambda r, c, s=0.1: (torch.randn(r, c, generator=g) * s).to(torch.bfloat16).to(gpu)
    one = lambda: torch.ones(d, device=gpu)
    t = {"embed": mat(V, d, 1.0), "lm_head": mat(V, d), "final_norm": one(),
         "layers": [{"attn_norm": one(), "w_qkv": mat((hq + 2 * hkv) * dh, d), "w_o": mat(d, hq * dh),
                     "ffn_norm": one(), "w_gate_up": mat(2 * ffn, d), "w_down": mat(d, ffn)}]}
    return engine.DeviceModel(engine.ModelShape(1, d, hq, hkv, dh, ffn, V, "bf16"), t, 1.0)


# (query heads, key/value heads, head_dim, prompt lengths, gen, block, mode, step kind)
CASES = [
    # shared tiles, blocks of eight (row group, head) pairs: ratio 1, 3, 7; rows of one
    # to seventeen groups, a last group of one row, a partly filled last block
    (32, 32, 128, [255, 1, 600, 17, 64], 64, 32, "none", "refresh"),
    (12, 4, 64, [1000, 513, 3], 40, 40, "none", "refresh"),
    (28, 4, 128, [1100, 33], 64, 64, "none", "refresh"),
    # shared tiles over short sequences, one block of 32 rows per head
    (32, 32, 128, [200], 64, 32, "dual", "cache"),
    (8, 8, 128, [1, 576], 64, 31, "dual", "cache"),
    # fewer keys than a tile
    (4, 4, 64, [5], 9, 9, "dual", "cache"),
    # per head, 32 rows and four key groups: several turns
    (8, 8, 128, [900, 641], 64, 32, "dual", "cache"),
    # per head, 64 rows and two key groups: grouped queries, multi-head
    (28, 4, 128, [400, 20, 130], 200, 64, "dual", "cache"),
    (32, 32, 128, [256], 256, 32, "none", "refresh"),
    # cache and recompute requests in one launch
    (32, 32, 128, [300, 40, 700, 128, 90, 511], 64, 32, "dual", "mixed"),
    (28, 4, 64, [300, 40, 700, 128], 64, 64, "dual", "mixed"),
]


# each kernel at the edges of its tiles, with the number that dlm_debug_attention_plan
# gives it
FORMS = [
    # grouped queries of at most 32 rows: two row groups x seven heads in two blocks
    (0, 28, 4, 128, [300, 31, 500, 1, 65, 64, 400, 129, 77, 700, 250, 33, 511, 40, 200], 48, 17,
     "dual", "cache"),
    # four-wave shared-tile blocks: more than two per CU, requests of one to four row groups
    (1, 32, 32, 64, [64 + 9 * i for i in range(17)], 64, 57, "dual", "cache"),
    # per head, 32 rows and four key groups: rows to a tile's edge, one turn and a row less
    (2, 8, 8, 128, [192], 64, 64, "none", "refresh"),
    (2, 4, 2, 64, [230, 191], 25, 25, "none", "refresh"),
    # per head, 32 rows and two key groups: an odd tile, fewer keys than a turn in one request
    (4, 8, 8, 64, [700, 1, 321], 33, 17, "dual", "cache"),
]


# keys split over blocks; the partials lie where the FFN's activations go, so the
# model's ffn is as wide as eight of them
SPLIT_CASES = [
    # more ranges than a short request has tiles (empty ranges), grouped queries
    (28, 4, 128, [2000, 3, 70], 64, 64, "dual", "cache"),
    # 17 tiles in ranges of three, the last tile of one key
    (32, 32, 128, [961], 64, 32, "dual", "cache"),
    # head_dim 64, a last block of one row, partly filled blocks
    (8, 2, 64, [700, 1], 57, 57, "dual", "cache"),
    # one row per head
    (4, 4, 128, [513], 1, 1, "dual", "cache"),
    # rows from the block to the end
    (28, 4, 128, [900], 200, 64, "prefix", "cache"),
    # three ranges over requests of very different lengths
    (32, 32, 128, [1500, 40, 700], 64, 32, "dual", "cache"),
]


@pytest.mark.parametrize("hq,hkv,dh,prompts,gen,block,mode,kind", CASES)
def test_attention_matches_fp64_on_its_inputs(gpu, hq, hkv, dh, prompts, gen, block, mode, kind):
    _check(gpu, hq, hkv, dh, prompts, gen, block, mode, kind, 64)


@pytest.mark.parametrize("kernel,hq,hkv,dh,prompts,gen,block,mode,kind", FORMS)
def test_each_kernel_matches_fp64_on_its_inputs(gpu, kernel, hq, hkv, dh, prompts, gen, block, mode,
                                                kind):
    lens = [p + gen for p in prompts]
    rows = lens if kind == "refresh" else [min(block, gen)] * len(lens)
    assert dlm.debug_attention_plan(hq, hkv, dh, rows, lens, 0) == (kernel, 1)
    _check(gpu, hq, hkv, dh, prompts, gen, block, mode, kind, 64)


@pytest.mark.parametrize("hq,hkv,dh,prompts,gen,block,mode,kind", SPLIT_CASES)
def test_split_keys_match_fp64_on_their_inputs(gpu, hq, hkv, dh, prompts, gen, block, mode, kind):
    ran = _check(gpu, hq, hkv, dh, prompts, gen, block, mode, kind, 16 * hq * (dh + 2))
    assert "attention_merge" in ran, ran


def _check(gpu, hq, hkv, dh, prompts, gen, block, mode, kind, ffn):
    """Checks one step's launch; returns the kernel classes that it ran."""
    model = _model(gpu, hq, hkv, dh, sum(prompts), ffn)
    eng = engine.Engine(model, len(prompts), max(prompts) + gen, mode)
    eng.cache_buf.view(torch.bfloat16).fill_(float("nan"))
    rng = np.random.default_rng(2)
    reqs = []
    for p in prompts:
        r = engine.Request(rng.integers(0, 64, p).astype(np.int32), gen, block, 0.9)
        eng.admit(r, 64)
        reqs.append(r)
    if kind != "refresh":
        eng.refresh(reqs)
        if kind == "mixed":
            reqs[0].refreshed_block = reqs[-1].refreshed_block = -1
    rows = eng.step_rows(reqs)
    dlm.profile_enable(model.handle, True)
    buf, _ = eng.debug_trace(reqs, 0, logits=False)
    torch.cuda.synchronize()
    classes = dlm.profile_read(model.handle)
    base = 0
    for r, (r0, r1) in zip(reqs, rows):
        n, L = r1 - r0, r.seq_len
        k, v = (x.double().numpy() for x in eng.read_kv(0, r.slot, L))
        q = buf["q"][base:base + n].double().cpu().numpy().reshape(n, hq, dh)
        got = buf["attn_out"][base:base + n].double().cpu().numpy().reshape(n, hq, dh)
        assert np.isfinite(got).all()
        for h in range(hq):
            kh, vh = k[:, h // (hq // hkv)], v[:, h // (hq // hkv)]
            s = q[:, h] @ kh.T / np.sqrt(dh)
            w = np.exp(s - s.max(1, keepdims=True))
            o = (w / w.sum(1, keepdims=True)) @ vh
            # two-term bf16 P and fp32 sums (as kernel_checks), the fp32 error of
            # the scores through the exponential, then the bf16 store
            mag = (np.abs(q[:, h]) @ np.abs(kh).T / np.sqrt(dh)).max()
            slack = (2.0 ** -15 + (L / 16 + 16 + 2 * dh / 32 * mag) * U) * np.abs(vh).max()
            err = half_ulp(np.abs(o) + slack, "bf16") + slack
            assert np.all(np.abs(got[:, h] - o) <= err), (r0, n, L, h)
        base += n
    return set(classes)
