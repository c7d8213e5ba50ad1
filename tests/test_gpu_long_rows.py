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


@pytest.mark.parametrize("V", [1000, 40000])
@pytest.mark.parametrize("temp", [1.0, 0.5])
def test_rows_of_minus_infinity_and_nan_at_a_temperature(V, temp):
    """-inf has no mass; a row without any finite value or with a NaN anywhere has no distribution: q is NaN, nothing is
    drawn (-1) and a draft tested against it is rejected."""
    amd = _amd()
    inf, nan = float("inf"), float("nan")
    q1 = torch.zeros((1, V), device="cuda")
    q1[0, 3] = 1.0
    row = torch.full((V,), -inf, device="cuda")
    row[3] = row[V - 2] = 1.5
    q, tok = amd.sample_row(row, temp, 1.0, 0.25)
    assert tok == 3 and q[3] == 0.5 and q[V - 2] == 0.5 and q.sum() == 1.0
    assert amd.accept_rows(row[None].contiguous(), q1, [3], [0.5], temp, 1.0, 0.5) == (1, -1)
    assert amd.accept_rows(row[None].contiguous(), q1, [3], [0.75], temp, 1.0, 0.5) == (0, V - 2)
    bad = [torch.full((V,), -inf, device="cuda"), row.clone(), row.clone(), torch.full((V,), nan, device="cuda")]
    bad[1][V // 2] = nan                # among -inf only: at 40000 ids a piece without any finite value
    bad[2][4] = nan
    for b in bad:
        q, tok = amd.sample_row(b, temp, 1.0, 0.25)
        assert tok == -1 and bool(q.isnan().all())
        assert amd.accept_rows(b[None].contiguous(), q1, [3], [0.0], temp, 1.0, 0.5) == (0, -1)
        assert amd.accept_rows(b[None].contiguous(), None, [], [], temp, 1.0, 0.5) == (0, -1)


@pytest.mark.parametrize("V", [32768, 32769, 50001, 131072, 540001])
@pytest.mark.parametrize("temp", [1.0, 0.0])
def test_a_distribution_may_replace_its_logits(V, temp):
    """q_out == logits, as a caller without a second row does it: the same q and token as with rows of their own."""
    amd = _amd()
    from paper_2408_11850_amd import binding
    lib = amd.load_library()
    for seed in range(4):
        row = torch.randn(V, generator=torch.Generator().manual_seed(seed * 7 + V)).mul_(3.0).cuda()
        q, tok = amd.sample_row(row, temp, 1.0, 0.3 + 0.1 * seed)
        out = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        amd.check(lib.spec_sample_row(binding._ptr(row), V, temp, 1.0, 0.3 + 0.1 * seed, binding._ptr(row), binding._ptr(out),
                                      binding._stream_ptr(torch.cuda.current_stream())))
        assert int(out.item()) == tok and torch.equal(row, q)


# a row in registers; pieces of 8192 ids: a last piece of one id, of an odd length, whole pieces (odd V: rows off every
# vector); 540001: more pieces than lanes
@pytest.mark.parametrize("V", [777, 32000, 32768, 32769, 33001, 40000, 65537, 131072, 540001])
@pytest.mark.parametrize("temp", [1.0, 0.7])
def test_a_draft_that_equals_the_target_is_never_rejected(V, temp):
    """q from sample_row and p inside accept_rows are the same bits for the same logits: r q[x] <= p[x] then holds up to
    the largest uniform, 1 - 2^-24, which one unit in the last place between p and q would already break."""
    amd = _amd()
    rows = torch.randn((32, V), generator=torch.Generator().manual_seed(V)).mul_(3.0).cuda()
    q = torch.empty_like(rows)
    x = []
    for i in range(32):
        q[i], tok = amd.sample_row(rows[i], temp, 1.0, (2 * i + 1) / 64.0)
        x.append(tok)
    assert amd.accept_rows(rows, q, x, [1.0 - 2.0 ** -24] * 32, temp, 1.0, 0.5) == (32, -1)
