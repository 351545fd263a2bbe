"""Polarized synthesis of several maps in one call against the same maps one by
one: the combination runs with the first launch over the polar caps (up to
three maps), later launches carry further maps' caps alone.  One and the same
arithmetic per map: 1e-13 of the map's scale.
"""
import pytest
import torch

from paper_1110_4874_amd.synthetic import alm_gaussian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N", [(3, 1), (65, 32), (300, 100), (511, 256)])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 7])
def test_maps_together_and_apart(gpu, L, N, n):
    p = gpu.Plan(L, N)
    E = torch.from_numpy(alm_gaussian(L - 1, list(range(60, 60 + n)))).cuda()
    B = torch.from_numpy(alm_gaussian(L - 1, list(range(90, 90 + n)))).cuda()
    out = torch.full((2, n, p.npix), float("nan"), dtype=torch.float64, device="cuda")
    p.pol_synthesis(E, B, out)
    assert bool(torch.isfinite(out).all())
    for b in range(n):
        one = torch.empty((2, 1, p.npix), dtype=torch.float64, device="cuda")
        p.pol_synthesis(E[:, b:b + 1].contiguous(), B[:, b:b + 1].contiguous(), one)
        scale = float(one.abs().max())
        assert float((out[:, b] - one[:, 0]).abs().max()) <= 1e-13 * scale
