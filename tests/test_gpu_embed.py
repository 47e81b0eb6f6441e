"""GPU check of the step's first kernel (embedding row, first norm): tables that are
not aligned to four values take one-value loads, and rows wider than 4096 are read
twice; both give the embedding's values exactly and the same norm bit for bit."""
import numpy as np
import pytest
import torch

from paper_2606_29094_amd import engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [128, 4096, 4160])
def test_unaligned_embedding_table(gpu, dtype, d):
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    V, dh, P, G = 37, 64, 21, 5
    g = torch.Generator().manual_seed(d)
    flat = torch.randn(V * d + 4, generator=g).to(dt)
    tok = np.random.default_rng(1).integers(0, V - 1, P).astype(np.int32)
    tok[3], tok[5] = -1, V                    # read as [MASK]
    one = 1 + torch.randn(d, generator=g).to(gpu) * 0.1
    z = lambda r, c: torch.zeros(r, c, dtype=dt, device=gpu)
    got = {}
    for off in (0, 1, 2, 3):
        buf = torch.empty(V * d + 4, dtype=dt, device=gpu)
        table = buf[off:off + V * d].view(V, d)
        table.copy_(flat[:V * d].view(V, d))
        assert table.data_ptr() % (4 * table.element_size()) == off * table.element_size()
        t = {"embed": table, "lm_head": z(V, d), "final_norm": one,
             "layers": [{"attn_norm": one, "w_qkv": z(3 * dh, d), "w_o": z(d, dh), "ffn_norm": one,
                         "w_gate_up": z(32, d), "w_down": z(d, 16)}]}
        model = engine.DeviceModel(engine.ModelShape(1, d, 1, 1, dh, 16, V, dtype), t, 1.0)
        eng = engine.Engine(model, 1, P + G, "none")
        r = engine.Request(tok, G, G, 0.9)
        eng.admit(r, V - 1)
        out, _ = eng.debug_trace([r], 0, logits=False)
        torch.cuda.synchronize()
        got[off] = out["h_in"].cpu(), out["a_attn"].cpu()
    ids = [v if 0 <= v < V else V - 1 for v in tok.tolist()] + [V - 1] * G
    rows = flat[:V * d].view(V, d)[ids].float()
    for h, a in got.values():
        assert torch.equal(h, rows)
        assert torch.equal(a, got[0][1])
    x = rows.double()
    want = x / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-5) * one.cpu().double()
    # d + 4 fp32 roundings of the sum, root, quotient and product; the store (bf16: eight
    # significant bits, half a unit of the last is at most 2^-8 of the value)
    tol = (d + 8) * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
    assert torch.all((got[0][1].double() - want).abs() <= tol * want.abs() + 1e-30)
