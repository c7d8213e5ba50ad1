"""Draws and acceptance of rows in registers, at the edges of the chunks their kernels are built for (run with -m gpu)."""
import numpy as np
import pytest
import torch

import synth
from oracle import sampling
from tests import test_gpu_long_rows as long_rows
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# 1, 2, 4 and 8 chunks of 4096 ids, one id to either side of each, rows that are no whole vectors
@pytest.mark.parametrize("V", [9, 1023, 4095, 4096, 4097, 8192, 8193, 12289, 16384, 16385, 24577, 28673, 32766])
@pytest.mark.parametrize("temp", [1.0, 0.0])
def test_rows_around_the_chunks(V, temp):
    long_rows.test_draws_and_acceptance_walk_rows_of_any_length(V, temp)


@pytest.mark.parametrize("V", [100, 4096, 4099, 16384, 30001])
def test_masked_ids_carry_no_mass(V):
    """Ids masked with -inf or the type's lowest value, at both ends and in whole chunks."""
    amd = long_rows._amd()
    row = synth.normal_tensor((V,), 3.0, 5, V, torch.float32)
    row[: V // 2] = float("-inf")
    row[V - 3:] = torch.finfo(torch.float32).min
    P = sampling.probs(row.numpy(), 1.0, 1.0)
    for u in (0.0, 0.4, 1.0 - 2.0 ** -24):
        q, tok = amd.sample_row(row.cuda(), 1.0, 1.0, u)
        np.testing.assert_allclose(q.cpu().numpy(), P, rtol=2e-5, atol=1e-12)
        assert V // 2 <= tok < V - 3 and P[tok] > 0
        n, y = amd.accept_rows(row[None].cuda(), None, [], [], 1.0, 1.0, u)
        assert n == 0 and y == tok
    assert amd.sample_row(row.cuda(), 0.0, 1.0, 0.5)[1] == int(row.argmax())
    row[:] = float("-inf")
    assert amd.sample_row(row.cuda(), 0.0, 1.0, 0.5)[1] == 0


@pytest.mark.parametrize("V", [9, 1000, 4096, 8191, 12000, 30001, 40000])
@pytest.mark.parametrize("temp,scale", [(float("inf"), 1.0), (1.0, -1.0)])
def test_multipliers_that_are_not_positive(V, temp, scale):
    """Infinite temperature is the uniform distribution, a negative scale turns a row round; no mass beyond the row."""
    amd = long_rows._amd()
    row = synth.normal_tensor((V,), 1.0, 6, V, torch.float32)
    z = row.double().numpy() * (0.0 if np.isinf(temp) else scale)
    P = np.exp(z) / np.exp(z).sum()
    for j in (0, V // 3, V - 1):
        u = float(np.float32(P[:j].sum() + 0.5 * P[j]))      # the middle of id j's share
        q, tok = amd.sample_row(row.cuda(), temp, scale, u)
        np.testing.assert_allclose(q.cpu().numpy(), P, rtol=2e-5, atol=1e-12)
        assert tok == j
        assert amd.accept_rows(row[None].cuda(), None, [], [], temp, scale, u) == (0, j)
    # a rejected draft: what p leaves beside a q that is all at id 1
    one = torch.zeros(1, V)
    one[0, 1] = 1.0
    W = P.copy()
    W[1] = 0.0
    W /= W.sum()
    j = V // 2
    u = float(np.float32(W[:j].sum() + 0.5 * W[j]))
    assert amd.accept_rows(row[None].cuda(), one.cuda(), [1], [0.999], temp, scale, u) == (0, j)


# 1, 2, 4 and 8 chunks in registers, and a long row
@pytest.mark.parametrize("V", [1000, 8192, 16000, 32000, 40000])
@pytest.mark.parametrize("temp", [1.0, 0.7])
def test_a_residual_without_mass_falls_back_to_the_target(V, temp):
    """q is p bit for bit but for a larger value at the draft, which is rejected: max(0, p - q) is 0 everywhere, not what a
    product loses when it is rounded, so the corrected token is the draw from p."""
    amd = long_rows._amd()
    row = synth.normal_tensor((V,), 3.0, 8, V, torch.float32).cuda()
    for u in (0.0, 0.11, 0.5, 0.83, 1.0 - 2.0 ** -24):
        q, want = amd.sample_row(row, temp, 1.0, u)
        q[V // 2] = 2.0
        assert amd.accept_rows(row[None], q[None], [V // 2], [0.999], temp, 1.0, u) == (0, want)
