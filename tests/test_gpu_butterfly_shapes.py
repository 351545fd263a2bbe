"""Compressed synthesis against the brute-force path on the same GPU, for each
group width of a pass (8, 4, 2 and 1 maps and sums of them) and both precisions
of the level products, at sizes whose skeletons leave lane groups partly filled.

Bars: the plan's ID tolerance plus 1e-12 of FP64 rounding; FP32 level products
round at 6e-8 over at most a few hundred terms a level: 2e-5.
"""
import numpy as np
import pytest
import torch

from paper_1110_4874_amd import sht
from paper_1110_4874_amd.synthetic import alm_gaussian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 3, 4, 5, 6, 8, 15, 17])
@pytest.mark.parametrize("L,N,levels", [(150, 64, 1), (333, 128, 2), (511, 200, 3)])
def test_group_widths(gpu, L, N, levels, B):
    alm = torch.from_numpy(alm_gaussian(L, list(range(40, 40 + B)))).cuda()
    p = gpu.Plan(L, N, 1e-11, max_levels=levels, store_fp32=True)
    ref = p.synthesis(alm, path=sht.PATH_BRUTE).cpu().numpy().reshape(B, -1)
    for prec, bar in ((sht.PREC_FP64, 1e-11 + 1e-12), (sht.PREC_FP32, 2e-5)):
        out = torch.full((B, p.npix), float("nan"), dtype=torch.float64, device="cuda")
        p.synthesis(alm, out, path=sht.PATH_BUTTERFLY, precision=prec)
        f = out.cpu().numpy()
        err = max(np.max(np.abs(f[b] - ref[b])) / np.max(np.abs(ref[b])) for b in range(B))
        assert err <= bar, (B, prec, err)
