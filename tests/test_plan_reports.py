"""Step counts that a plan reports, against the chains it holds: the steps in
double-double and the lane-steps of the Legendre kernel's blocks.  Host-only."""
import pytest

DEAD = 0x3FFFFFFF


def lane_steps(p, bounds, R):
    """bounds: (first group, end, groups a block) of each part."""
    L, north = p.L, 2 * p.nside
    total = 0
    for m in range(L + 1):
        lo = []
        for g in range((north + 63) // 64):
            s = [p.start(m, t, k)[0] for t in (0, 1) for k in range(64 * g, min(64 * g + 64, north))]
            lo.append(min(s))
        for g0, g1, w in bounds:
            for b in range(g0, g1, w):
                groups = lo[b:min(b + w, g1)]
                for t in (0, 1):
                    n = (L - m - t) // 2 + 1 if m + t <= L else 0
                    if min(groups) < n:
                        total += 64 * len(groups) * ((n - min(groups) + 7) // 8 * 8)
    return total


# (L, nside, threshold) -> parts: split groups, or double-double ones, then the plain ones
@pytest.mark.parametrize("L,N,dd_sin,parts,dd", [
    (40, 100, None, [(0, 4, 2)], False),
    (300, 150, None, [(0, 1, 2), (1, 5, 2)], False),       # split: sin at the end of group 0 is 0.34, of group 1 0.68
    (300, 300, None, [(0, 2, 2), (2, 10, 2)], False),      # 0.17 and 0.34
    (300, 150, 0.4, [(0, 2, 1), (2, 5, 2)], True),         # double-double: 72 rings
    (300, 150, 0.0, [(0, 5, 2)], False),
    (1400, 40, None, [(0, 1, 1), (1, 2, 2)], True),        # reaches too far from the pole
])
def test_step_counts(L, N, dd_sin, parts, dd):
    from paper_1110_4874_amd import sht
    p = sht.Plan(L, N, dd_sin=dd_sin, host_only=True)
    info = p.info()
    assert (info["n_step_dd"] > 0) == dd
    assert info["n_step_dd"] <= info["n_step_exec"]
    if L <= 300:
        assert info["n_step_lanes"] == lane_steps(p, parts, 2)
