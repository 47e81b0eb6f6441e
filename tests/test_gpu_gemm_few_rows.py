"""GPU checks of the GEMM tiles that serve launches of up to 1024 rows, through
the C ABI (dlm_debug_gemm): the rotated K walk (one row tile and weight rows a
power of two apart) of every tile configuration, at the smallest and largest row
count of its tile, against the fp64 product of the same operands."""
import numpy as np
import pytest
import torch

from kernel_checks import gemm_tol
from paper_2606_29094_amd import dlm

pytestmark = pytest.mark.gpu

CONFIGS = [(cfg,) + dlm.debug_gemm_info(cfg)[:2] for cfg in range(128) if dlm.debug_gemm_info(cfg)]


@pytest.mark.parametrize("cfg,bm,bn", CONFIGS, ids=lambda v: str(v))
def test_rotated_k_walk_matches_fp64_product(gpu, cfg, bm, bn):
    # K = 2048: weight rows 4 KB apart, the smallest pitch that rotates; more
    # column tiles than the 4 k-tiles of an 8-way slice, so the start wraps
    N, K = 6 * bn + 48, 2048
    g = torch.Generator().manual_seed(cfg)
    b = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16)
    for M in (1, bm - 5, bm):
        a = (torch.randn(M, K, generator=g) * 0.5).to(torch.bfloat16)
        A, B = a.double().numpy(), b.double().numpy()
        for s in (1, 8):
            c = torch.full((s, M, N) if s > 1 else (M, N), float("nan"), device=gpu)
            dlm.debug_gemm(cfg, 0, a.to(gpu), b.to(gpu), c, splits=s)
            c = c.cpu().double().numpy().reshape(s, M, N)
            w = K // s
            for z in range(s):
                x, y = A[:, z * w:(z + 1) * w], B[:, z * w:(z + 1) * w]
                # one rounding per 32-product step in any order of the steps
                assert np.all(np.abs(c[z] - x @ y.T) <= gemm_tol(x, y, 1, "bf16")), (cfg, M, s, z)
