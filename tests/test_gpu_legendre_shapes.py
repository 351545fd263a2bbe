"""Legendre phase over its wave shapes: rings per lane, maps per pass and the
ring groups of the split recurrence near the poles.

Every shape is compared with the long-double oracle on sampled rings (poles,
64-ring group edges, the equator) at the brute-force bar of 1e-12 relative to
the largest phase: the recurrence's own error is below 1e-13 at these sizes.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1110_4874_amd.synthetic import alm_gaussian

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _err(p, alm, rings):
    q = p.legendre_phase(torch.from_numpy(alm).cuda()).cpu().numpy()
    ref = oracle.legendre_phase_rings(p.L, p.nside, alm, np.array(rings), ld=True)
    return np.max(np.abs(q[np.array(rings) - 1] - ref)) / np.max(np.abs(ref))


# chain lengths at and around the 8-step chunk; 1, 2, 3 and 5 ring groups, full and partial
@pytest.mark.parametrize("L,N", [(7, 4), (16, 32), (33, 33), (127, 64), (128, 65), (250, 130)])
@pytest.mark.parametrize("R", [1, 2, 4])
def test_rings_per_lane_and_maps(gpu, L, N, R):
    p = gpu.Plan(L, N, rings_per_lane=R)
    rings = sorted({k for k in (1, 2, 63, 64, 65, 128, 129, 2 * N - 1, 2 * N, 2 * N + 1, 4 * N - 1) if k < 4 * N})
    for B in (1, 2, 3, 4, 5, 6, 7, 8, 11):
        err = _err(p, alm_gaussian(L, list(range(B))), rings)
        assert err <= TOL, (L, N, R, B, err)


# the split recurrence: one partial group (few rings), groups past the
# threshold, and a plan whose polar group reaches too far for it
@pytest.mark.parametrize("L,N,R", [(300, 150, 1), (700, 400, 2), (900, 512, 4), (1400, 40, 1)])
def test_polar_groups(gpu, L, N, R):
    p = gpu.Plan(L, N, rings_per_lane=R)
    n_dd = p.info()["n_dd_rings"]
    assert n_dd > 0
    rings = sorted({k for k in (1, 2, 3, n_dd, n_dd + 1, 63, 64, 65, 100, 128, 129, 192, 193, N, 2 * N, 4 * N - 2, 4 * N - 1)
                    if 0 < k < 4 * N})
    for B in (1, 3, 8):
        alm = alm_gaussian(L, list(range(B)), spectrum="white")
        err = _err(p, alm, rings)
        dd = gpu.Plan(L, N, dd_sin=0.1 * L / 4095.0, rings_per_lane=R)  # the same rings, in double-double
        err_dd = _err(dd, alm, rings)
        print(f"L={L} N={N} B={B}: {err:.2e}, double-double {err_dd:.2e}")
        assert err <= TOL and err_dd <= TOL, (B, err, err_dd)


# the adjoint's waves: one and two ring groups a wave, passes of 1 to 8 maps,
# polar groups (even and odd numbers), more groups than one launch covers
@pytest.mark.parametrize("L,N", [(7, 4), (33, 33), (127, 64), (250, 130), (300, 150), (700, 400)])
@pytest.mark.parametrize("R", [0, 1, 2])
def test_adjoint_rings_per_wave_and_maps(gpu, L, N, R):
    p = gpu.Plan(L, N, rings_per_lane=R)
    y = np.random.default_rng(L + N).standard_normal((11, 12 * N * N))
    ref = oracle.adjoint(L, N, y)
    for B in (1, 2, 3, 4, 5, 6, 8, 11) if L < 700 else (1, 3, 11):
        g = p.adjoint(torch.from_numpy(y[:B]).cuda()).cpu().numpy()
        err = np.max(np.abs(g - ref[:, :B])) / np.max(np.abs(ref))
        assert err <= TOL, (L, N, R, B, err)


def test_adjoint_over_several_launches(gpu):
    # 20 and 36 ring groups, one a wave: 16 groups per launch, added in place
    for L, N, R in ((60, 640, 1), (40, 1152, 2)):
        y = np.random.default_rng(N).standard_normal((3, 12 * N * N))
        ref = oracle.adjoint(L, N, y)
        for dd in (None, 0.05):  # 0.05: the first groups in double-double
            p = gpu.Plan(L, N, rings_per_lane=R, dd_sin=dd)
            g = p.adjoint(torch.from_numpy(y).cuda()).cpu().numpy()
            err = np.max(np.abs(g - ref)) / np.max(np.abs(ref))
            assert err <= TOL, (L, N, dd, err)
