"""The adjoint does not depend on rings_per_lane, which is the synthesis kernel's
(the order of its sums, and so the last bits, would show that it does)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,B", [(90, 64, 3), (120, 300, 2), (60, 640, 4), (200, 450, 7)])
def test_same_bits_for_any_rings_per_lane(gpu, L, N, B):
    y = torch.from_numpy(np.random.default_rng(L).standard_normal((B, 12 * N * N))).cuda()
    ref = gpu.Plan(L, N).adjoint(y)
    for R in (1, 2, 4):
        assert torch.equal(gpu.Plan(L, N, rings_per_lane=R).adjoint(y), ref), R
