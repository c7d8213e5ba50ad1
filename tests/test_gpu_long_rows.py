"""Vocabulary rows beyond the registers of one workgroup: pieces of 8192 ids (run with -m gpu)."""
import numpy as np
import pytest
import torch

import synth
from oracle import sampling
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _amd():
    import paper_2408_11850_amd as amd
    amd.load_library()
    return amd


# 32767 .. 32769: registers or pieces; 40961: a piece of one id; 65535, 65537: misaligned rows; 131072: whole pieces
@pytest.mark.parametrize("V", [32767, 32768, 32769, 40961, 65535, 65537, 131072])
@pytest.mark.parametrize("temp", [1.0, 0.0])
def test_draws_and_acceptance_walk_rows_of_any_length(V, temp):
    amd = _amd()
    rows = synth.normal_tensor((4, V), 3.0, 5, V, torch.float32)
    rows[1] = -1000.0                                 # one id carries all the mass, in the last piece
    rows[1, V - 1] = 5.0
    us = [0.0, 0.5, 1.0 - 2.0 ** -24, 0.123]
    P = [sampling.probs(r.numpy(), temp, 1.0) for r in rows]
    drafts = []
    for i in range(4):
        q, tok = amd.sample_row(rows[i].cuda(), temp, 1.0, us[i])
        q = q.cpu().numpy()
        np.testing.assert_allclose(q, P[i], rtol=2e-5, atol=1e-12)
        cdf = np.cumsum(q.astype(np.float64))
        want = int(np.searchsorted(cdf, us[i] * cdf[-1], side="right"))
        assert q[tok] > 0 and (tok == want or np.min(np.abs(cdf / cdf[-1] - us[i])[q > 0]) <= 1e-9)
        drafts.append(tok)
    # p == q: everything accepted, the bonus token drawn from the fourth row (three rows tested)
    Q = torch.from_numpy(np.stack(P[:3]).astype(np.float32)).cuda()
    n, y = amd.accept_rows(rows.cuda(), Q, drafts[:3], [0.5] * 3, temp, 1.0, us[3])
    assert (n, y) == (3, drafts[3])
    # a draft the target gives no mass, in the second row: rejected, the corrected token is that row's only id
    bad = torch.zeros((2, V), device="cuda")
    bad[0] = Q[0]
    bad[1, 7] = 1.0
    n, y = amd.accept_rows(rows[:2].contiguous().cuda(), bad, [drafts[0], 7], [0.5, 0.5], temp, 1.0, 0.7)
    assert (n, y) == (1, V - 1)


@pytest.mark.parametrize("V", [1000, 40000])
def test_greedy_rows_of_the_lowest_value_and_nan(V):
    """The lowest id of the largest value that is a number; rows of -inf give id 0."""
    amd = _amd()
    row = torch.full((V,), float("-inf"), device="cuda")
    assert amd.sample_row(row, 0.0, 1.0, 0.5)[1] == 0
    row[:] = float("nan")
    row[5] = row[V - 3] = -2.0
    assert amd.sample_row(row, 0.0, 1.0, 0.5)[1] == 5
    assert amd.accept_rows(row[None].contiguous(), None, [], [], 0.0, 1.0, 0.5) == (0, 5)
