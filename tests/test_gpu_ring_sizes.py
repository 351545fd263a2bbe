"""Ring stage over its transform sizes, both directions: every power of two
from 2 to 4096 and Bluestein lengths at the edges of each padded size, against
the ring sums by definition (tests/ring_defs.py).  The transforms take at most
24 radix-2 stages of a few roundings each, so errors stay near 1e-15 of the
largest value; the bar is that of the other ring tests, 1e-12.
"""
import numpy as np
import pytest
import torch

import oracle
from ring_defs import ring_direct, ring_direct_adjoint

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _rings(N):
    ks = {1, 2, 3, N - 1, N, N + 1, 2 * N, 3 * N, 3 * N + 1, 4 * N - 3, 4 * N - 1}
    for e in range(12):  # polar ring k: n = 2 k points, Bluestein halves of k padded past 2 k - 1
        ks |= {k for k in (2 ** e - 1, 2 ** e, 2 ** e + 1, 3 * 2 ** e) if k < N}
    return sorted(k for k in ks if 0 < k < 4 * N)


@pytest.mark.parametrize("L,N,B", [(9, 1, 1), (40, 2, 3), (33, 5, 2), (50, 16, 1), (300, 33, 4), (70, 64, 2), (130, 100, 8),
                                   (600, 128, 1), (45, 257, 3), (80, 500, 4), (24, 1024, 2), (20, 1500, 1), (17, 2000, 2),
                                   (12, 2048, 3)])
def test_every_transform_size(gpu, L, N, B):
    rng = np.random.default_rng(N)
    nr, npix = 4 * N - 1, 12 * N * N
    p = gpu.Plan(L, N)
    q = torch.view_as_complex(torch.from_numpy(rng.standard_normal((nr, L + 1, B, 2))).cuda())
    y = torch.from_numpy(rng.standard_normal((B, npix))).cuda()
    f = torch.full((B, npix), float("nan"), dtype=torch.float64, device="cuda")
    p.ring_synthesis(q, out=f)
    g = p.ring_analysis(y)
    assert bool(torch.isfinite(f).all()) and bool(torch.isfinite(torch.view_as_real(g)).all())
    worst = 0.0
    for ring in _rings(N):
        z, st, J, s, off = oracle.ring_info(N, ring)
        ref = ring_direct(q[ring - 1].cpu().numpy(), J, s)
        worst = max(worst, np.max(np.abs(f[:, off:off + J].cpu().numpy() - ref)) / np.max(np.abs(ref)))
        ref = ring_direct_adjoint(y[:, off:off + J].cpu().numpy(), L, J, s, 2.0)
        worst = max(worst, np.max(np.abs(g[ring - 1].cpu().numpy() - ref)) / np.max(np.abs(ref)))
    print(f"L={L} N={N} B={B}: {worst:.2e}")
    assert worst <= TOL
