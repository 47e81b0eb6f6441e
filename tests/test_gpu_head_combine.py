"""GPU check of the fused head's combine over vocabulary tiles at the row counts
where its form changes (one row per block below 1024 rows, 16 rows per block
from there) and where its last block is partly filled, against fp64 on the same
rows: confidences, and predictions with the lowest id on exact ties."""
import pytest
import torch

from paper_2606_29094_amd import dlm, engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows", [1, 3, 255, 1023, 1024, 1025, 1039])
def test_head_combine_over_row_counts(gpu, dtype, rows):
    d, V = 128, 4999                      # 40 vocabulary tiles of 128, the last one ragged
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(rows)
    w = torch.randn(V, d, generator=g).to(dt)
    w[4000] = w[17]                       # an exact tie across tiles
    u = torch.randn(rows, d, generator=g).to(dt)
    u[0] = w[17]
    one = torch.ones(d, device=gpu)
    z = lambda r, c: torch.zeros(r, c, dtype=dt, device=gpu)
    t = {"embed": z(V, d), "lm_head": w.to(gpu), "final_norm": one,
         "layers": [{"attn_norm": one, "w_qkv": z(3 * d, d), "w_o": z(d, d), "ffn_norm": one,
                     "w_gate_up": z(128, d), "w_down": z(d, 64)}]}
    model = engine.DeviceModel(engine.ModelShape(1, d, 2, 2, 64, 64, V, dtype), t, 0.25)
    ws = torch.empty(dlm.workspace_bytes(model.handle, max(rows, 64), 64), dtype=torch.uint8,
                     device=gpu)
    conf = torch.full((rows,), -1.0, device=gpu)
    tok = torch.full((rows,), -1, dtype=torch.int32, device=gpu)
    dlm.head_confidence(model.handle, u.to(gpu), rows, conf, tok, ws)
    zz = (u.double() @ w.double().T) * 0.25
    p = torch.softmax(zz, 1)
    top, at = p.max(1)
    # |z| <= ~100: fp32 products and sums (d + 2 roundings) move z by < 1e-4
    assert torch.all((conf.cpu().double() / top - 1).abs() < 1e-3)
    gap = zz.topk(2, 1).values
    clear = gap[:, 0] - gap[:, 1] > 1e-3
    assert torch.equal(tok.cpu()[clear].long(), at[clear])
    assert int(tok[0]) == 17
