"""Rings near the equator, the double root of the two-step recurrence in z^2,
where its rounding errors add up most: the Legendre phase is no further from
double-double than the same recurrence evaluated in FP64 as App. A.2 writes it
(coefficients beta, alpha beta, gamma, each rounded once; fused multiply-adds)."""
import numpy as np
import pytest
import torch

from paper_1110_4874_amd.synthetic import alm_gaussian

pytestmark = pytest.mark.gpu
ld = np.longdouble


def fp64_phase(p, m, z, alm):
    """q_m at the north rings z (index, z) by the unscaled recurrence in FP64."""
    ks, z2 = z
    off = m * (2 * p.L + 3 - m) // 2
    coef = p.coef(m)  # beta, alpha beta, gamma at l = m ..
    parts = []
    for t in (0, 1):
        n = (p.L - m - t) // 2 + 1
        starts = [p.start(m, t, int(k)) for k in ks]
        p0, p1 = np.zeros(len(ks)), np.zeros(len(ks))
        acc = np.zeros((len(ks), alm.shape[1]), dtype=np.complex128)
        for i in range(n):
            for j, (i0, v) in enumerate(starts):
                if i0 == i:
                    p0[j], p1[j] = v
            acc += p0[:, None] * alm[off + t + 2 * i][None]
            if t + 2 * i + 2 < len(coef):
                b, ab, g = coef[t + 2 * i + 2]
                a = (ld(b) * z2 + ld(ab)).astype(np.float64)
                p0, p1 = p1, (ld(1) * a * p1 + g * p0).astype(np.float64)
        parts.append(acc)
    return parts[0] + parts[1]


@pytest.mark.parametrize("L,N", [(300, 150), (1023, 512)])
def test_no_further_off_than_the_plain_recurrence(gpu, L, N):
    p, exact = gpu.Plan(L, N), gpu.Plan(L, N, dd_sin=10.0)
    alm = alm_gaussian(L, [7, 8], spectrum="white")
    a = torch.from_numpy(alm).cuda()
    k = np.arange(2 * N - N // 8, 2 * N)[::4]  # north rings near the equator, and the equator
    q, ref = (x.legendre_phase(a).cpu().numpy()[k] for x in (p, exact))
    z2 = ((4 * N - 2 * (k + 1)) / ld(3 * N)) ** 2
    z2 = z2.astype(np.float64)
    ours, plain = 0.0, 0.0
    for m in range(0, int(0.9 * L), max(1, L // 128)):
        f = fp64_phase(p, m, (k, z2), alm)
        if m == 0:
            f = f.real + 0j
        ours += np.sum(np.abs(q[:, m] - ref[:, m]) ** 2)
        plain += np.sum(np.abs(f - ref[:, m]) ** 2)
    print(f"L={L}: {np.sqrt(ours):.3e}, unscaled FP64 {np.sqrt(plain):.3e}")
    assert ours <= plain
