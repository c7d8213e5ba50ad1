"""A row of a forward over up to 8 tokens has the same bits however many rows follow it (run with -m gpu)."""
import numpy as np
import pytest

import synth
from tests.test_gpu_stale_cache import model
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def assert_rows_share_their_bits(s, max_seq, lengths):
    import paper_2408_11850_amd as amd
    m = model(s, 3)
    ids = synth.prompt_tokens(max_seq, s.vocab, 7).tolist()
    ctx = amd.SpecContext(m, m, gamma_max=8, max_seq=max_seq)
    for n in lengths:
        ctx.prefill(ids[:n], which_mask=1)
        rows = ctx.verify(ids[n - 1:n + 7], want_logits=True).copy()
        assert np.isfinite(rows).all() and rows.std() > 0.1
        for k in range(1, 8):
            ctx.rollback_kv(amd.SPEC_TARGET, n - 1)
            got = ctx.verify(ids[n - 1:n - 1 + k], want_logits=True)
            assert np.array_equal(got, rows[:k]), (n, k)
    ctx.close()


# the attention, behind narrow projections: room for 320 .. 1024 positions with any grouping, for 1280 with up to 16 query rows
# (there the split count follows the number of 16-row tiles)
@pytest.mark.parametrize("heads,kv,dh,max_seq", [(h, k, d, n) for n in (256, 448, 900, 1200)
                                                 for h, k, d in ((2, 2, 128), (4, 2, 64), (8, 1, 128)) if n < 1024 or h <= 2 * k])
def test_attention_rows(heads, kv, dh, max_seq):
    assert_rows_share_their_bits(synth.ModelShape(2, 256, heads, kv, 512, 1008, head_dim=dh), max_seq, (40, 200, max_seq - 20))


# the projections: QKV, O, gate/up, down and LM head of one half to eight panels per CU, short ranges of K and long ones (the
# plans behind them are compared on the host, over a grid of shapes, in test_abi.py)
@pytest.mark.parametrize("d,heads,ffn,vocab", [(2048, 16, 5504, 32000), (4096, 32, 11008, 16384), (8192, 4, 3072, 10240),
                                               (7168, 56, 2048, 20496)])
def test_projection_rows(d, heads, ffn, vocab):
    assert_rows_share_their_bits(synth.ModelShape(2, d, heads, heads, ffn, vocab, head_dim=128), 256, (100,))
