"""GPU checks of the fp32 model's kernels at the sizes where their tiles end:
attention (16 query rows per block, 32-key groups dealt to the waves) and the
small-tile GEMM (16 x 32 outputs, 16-wide k groups dealt to eight waves), each
on exactly the values the kernel received (dlm_debug_trace), against fp64. The
cache holds NaN wherever no step wrote, so a read past a sequence shows."""
import numpy as np
import pytest
import torch

from paper_2606_29094_amd import engine

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def _model(gpu, hq, hkv, dh, d, ffn, seed):
    g = torch.Generator().manual_seed(seed)
    mat = lambda r, c: (torch.randn(r, c, generator=g) * 0.05).to(gpu)
    one = lambda: torch.ones(d, device=gpu)
    t = {"embed": (torch.randn(97, d, generator=g)).to(gpu), "lm_head": mat(97, d),
         "final_norm": one(),
         "layers": [{"attn_norm": one(), "w_qkv": mat((hq + 2 * hkv) * dh, d),
                     "w_o": mat(d, hq * dh), "ffn_norm": one(), "w_gate_up": mat(2 * ffn, d),
                     "w_down": mat(d, ffn)}]}
    shape = engine.ModelShape(1, d, hq, hkv, dh, ffn, 97, "f32")
    return engine.DeviceModel(shape, t, 1.0), t


def _gemm_ok(got, a, w, extra=0.0):
    """a, w: the fp32 operands. K products and K sums, each rounded once, in any order."""
    a, w = a.double().cpu().numpy(), w.double().cpu().numpy()
    ref, mag = a @ w.T, np.abs(a) @ np.abs(w).T
    tol = (a.shape[1] + 2) * U * (mag + np.abs(extra)) + U * np.abs(extra)
    return ref, np.abs(got.double().cpu().numpy() - (ref + extra)) <= tol


# lengths at the edges of the 16-row tiles, 32-key groups, and the 128 keys of
# one turn of the waves; the last two turn more than once
@pytest.mark.parametrize("hq,hkv,dh,ffn", [(4, 4, 64, 688), (6, 2, 128, 48), (1, 1, 64, 16)])
@pytest.mark.parametrize("lens", [(1,), (15, 17), (16, 31, 33), (127, 129), (32, 300, 64)])
def test_fp32_kernels_match_fp64_on_their_inputs(gpu, hq, hkv, dh, ffn, lens):
    d = 192
    model, t = _model(gpu, hq, hkv, dh, d, ffn, seed=sum(lens))
    eng = engine.Engine(model, len(lens), max(lens), "none")
    eng.cache_buf.view(torch.float32).fill_(float("nan"))
    rng = np.random.default_rng(1)
    reqs = []
    for L in lens:
        n = min(L, 8)
        r = engine.Request(rng.integers(0, 96, L - n).astype(np.int32), n, n, 0.9)
        eng.admit(r, 96)
        reqs.append(r)
    buf, splits = eng.debug_trace(reqs, 0, logits=False)
    torch.cuda.synchronize()
    w = t["layers"][0]
    ref, ok = _gemm_ok(buf["qkv"].double().sum(0), buf["a_attn"], w["w_qkv"])
    assert ok.all()
    row = 0
    for r, L in zip(reqs, lens):
        k, v = (x.double().numpy() for x in eng.read_kv(0, r.slot, L))
        q = buf["q"][row:row + L].double().cpu().numpy().reshape(L, hq, dh)
        got = buf["attn_out"][row:row + L].double().cpu().numpy().reshape(L, hq, dh)
        for h in range(hq):
            s = q[:, h] @ k[:, h // (hq // hkv)].T / np.sqrt(dh)
            p = np.exp(s - s.max(1, keepdims=True))
            o = (p / p.sum(1, keepdims=True)) @ v[:, h // (hq // hkv)]
            # score error (dh products) through the exponential, then L weighted sums
            mag = np.abs(q[:, h]) @ np.abs(k[:, h // (hq // hkv)]).T / np.sqrt(dh)
            tol = ((2 * (dh + 2) * mag.max(1) + L + 16) * U)[:, None] * np.abs(v).max()
            assert np.all(np.abs(got[:, h] - o) <= tol), (L, h)
        row += L
    _, ok = _gemm_ok(buf["h_mid"], buf["attn_out"], w["w_o"], buf["h_in"].double().cpu().numpy())
    assert ok.all()
    _, ok = _gemm_ok(buf["h_out"], buf["act"], w["w_down"], buf["h_mid"].double().cpu().numpy())
    assert ok.all()
    y = (buf["a_ffn"].double() @ w["w_gate_up"].double().T).cpu().numpy()
    want = y[:, :ffn] / (1 + np.exp(-y[:, :ffn])) * y[:, ffn:]
    mag = (buf["a_ffn"].double().abs() @ w["w_gate_up"].double().abs().T).cpu().numpy()
    e = (d + 2) * U * mag
    slack = 1.1 * e[:, :ffn] * np.abs(y[:, ffn:]) + np.abs(y[:, :ffn]) * e[:, ffn:] \
        + e[:, :ffn] * e[:, ffn:] + 16 * U * np.abs(want)
    assert np.all(np.abs(buf["act"].double().cpu().numpy() - want) <= slack)


@pytest.mark.parametrize("far", [(0, 32), (32, 64), (96, 224), (128, 256)])
def test_fp32_key_group_whose_scores_overflow(gpu, far):
    """Keys whose scores overflow to -inf get weight 0, also where they fill the
    first 32-key group that a wave reads (the waves take the groups in turn)."""
    d = dh = 64
    L = 300
    t = {"embed": torch.zeros(97, d), "lm_head": torch.zeros(97, d)}
    t["embed"][:, 0] = 1.0                    # every token: q[31] of 5e19 to 8e19
    t["embed"][1, 1] = 1.0                    # token 1: k[31] of about -6e19, scores of -inf
    t["embed"][:, 2] = torch.linspace(-1, 1, 97)
    w = torch.zeros(3 * dh, d)
    w[31, 0], w[dh + 31, 1] = 1e19, -1e19     # the last rotary pair: its angle is 0 at every position
    w[2 * dh:, 2] = torch.linspace(0.1, 1.0, dh)
    one = torch.ones(d, device=gpu)
    z = lambda r, c: torch.zeros(r, c, device=gpu)
    dev = {k: v.to(gpu) for k, v in t.items()}
    dev["final_norm"] = one
    dev["layers"] = [{"attn_norm": one, "w_qkv": w.to(gpu), "w_o": z(d, dh), "ffn_norm": one,
                      "w_gate_up": z(32, d), "w_down": z(d, 16)}]
    shape = engine.ModelShape(1, d, 1, 1, dh, 16, 97, "f32", rope_theta=1e37)
    model = engine.DeviceModel(shape, dev, 1.0)
    eng = engine.Engine(model, 1, L, "none")
    tok = np.arange(2, 2 + L).astype(np.int32) % 90 + 2
    tok[far[0]:far[1]] = 1
    r = engine.Request(tok[:L - 8], 8, 8, 0.9)
    eng.admit(r, 96)
    buf, _ = eng.debug_trace([r], 0, logits=False)
    torch.cuda.synchronize()
    k, v = (x.double().numpy()[:, 0] for x in eng.read_kv(0, r.slot, L))
    q = buf["q"].double().cpu().numpy()
    s = q @ k.T / np.sqrt(dh)
    assert (s[:, far[0]:far[1]] < -1e38).all()          # -inf in fp32
    assert np.abs(s[:, [i for i in range(L) if not far[0] <= i < far[1]]]).max() == 0
    p = np.exp(s - s.max(1, keepdims=True))
    o = (p / p.sum(1, keepdims=True)) @ v
    got = buf["attn_out"].double().cpu().numpy()
    # equal weights: L sums and products of fp32 values
    assert np.all(np.abs(got - o) <= (L + 16) * U * np.abs(v).max())
