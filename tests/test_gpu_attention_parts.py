"""Decode attention with the columns of a head dealt to four, two and one workgroups (run with -m gpu)."""
import pytest

import synth
from oracle import transformer
from tests.test_gpu_forward import LOGIT_TOL, _custom, _rel_err, _setup
from tests.test_gpu_row_bits import assert_rows_share_their_bits
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# On 256 CUs four workgroups up to 64 of KV heads x 16-row tiles, two up to 128.  Rows M x heads per KV head: with 4 of them the
# second tile starts at M = 5, so a forward over 1 .. 8 tokens takes four and two (40 KV heads), or two and one (72).
SHAPES = [(160, 40, 128), (160, 40, 64), (288, 72, 64)]


@pytest.mark.parametrize("heads,kv,dh", SHAPES)
def test_rows_keep_their_bits_between_the_parts(heads, kv, dh):
    assert_rows_share_their_bits(synth.ModelShape(2, 256, heads, kv, 512, 1008, head_dim=dh), 448, (40, 300))


@pytest.mark.parametrize("heads,kv,dh", SHAPES)
def test_parts_against_the_oracle(heads, kv, dh):
    cfg = _custom(synth.ModelShape(2, 256, heads, kv, 512, 1008, head_dim=dh), 1)
    cfg.n_prompt = 300
    amd, ctx, tm, _ = _setup(cfg, gamma_max=15)
    ids = synth.prompt_tokens(400, 1008, 7).tolist()
    for context in (0, 33, 250):
        ctx.prefill(ids[:context + 1])
        ocm = transformer.CachedModel(tm, 400)
        if context:
            ocm.feed(ids[:context])
        ref = ocm.feed(ids[context:context + 16])
        for m in (1, 4, 5, 16):
            assert _rel_err(ctx.verify(ids[context:context + m], want_logits=True), ref[:m]) <= LOGIT_TOL, (context, m)
            ctx.rollback_kv(amd.SPEC_TARGET, context)
        ctx.verify(ids[context:context + 5])
        got = ctx.verify(ids[context + 5:context + 8], want_logits=True)
        assert _rel_err(got, ref[5:8]) <= LOGIT_TOL, context
    ctx.close()
