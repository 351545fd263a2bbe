"""The host evaluations of a chain read its n_t values: an x with fewer ends in
zeros, and nothing behind it is read."""
import numpy as np
import pytest


@pytest.mark.parametrize("form", ["butterfly", "interp"])
def test_short_x_is_zero_extended(form):
    from paper_1110_4874_amd import sht
    p = sht.Plan(63, 32, 1e-10 if form == "butterfly" else 0.0, host_only=True, interp=form == "interp")
    apply = p.butterfly_apply_host if form == "butterfly" else p.interp_apply_host
    behind = np.full(64, 1e30)
    behind[:20] = np.random.default_rng(3).standard_normal(20)
    for m, t in ((0, 0), (3, 1), (20, 0)):
        whole = np.zeros((63 - m - t) // 2 + 1)
        whole[:20] = behind[:20]
        assert np.array_equal(apply(m, t, behind[:20]), apply(m, t, whole))
