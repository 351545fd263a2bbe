"""Device memory of a plan: the unscaled recurrence coefficients, high and low
parts, are held by the plans whose kernels read them, and by no others."""
import pytest

pytestmark = pytest.mark.gpu


def test_coefficient_tables(gpu):
    L, N = 500, 300
    table = 32 * sum((L - m + 1 + 24 + 1) // 2 * 2 for m in range(L + 1))  # bytes: four doubles an entry
    plain, dd = (gpu.Plan(L, N, dd_sin=d).info() for d in (0.0, 0.3))
    assert plain["n_dd_rings"] == 0 and dd["n_dd_rings"] > 0
    assert dd["device_bytes"] - plain["device_bytes"] >= 2 * table  # high and low parts (and the starts' low parts)
