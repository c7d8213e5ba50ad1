"""Decode attention of few query rows over a context of 449..1024 positions (run with -m gpu)."""
import pytest

import synth
from oracle import transformer
from tests.test_gpu_forward import LOGIT_TOL, _custom, _rel_err, _setup
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# up to 8 query rows per KV head take 16 waves, more of them 8; contexts around a chunk, a page, one round of 15 chunks (480
# positions) and two, and the last position there is room for
@pytest.mark.parametrize("heads,kv,dh", [(2, 2, 128), (4, 2, 64), (8, 1, 128)])
def test_contexts_around_the_rounds_of_sixteen_waves(heads, kv, dh):
    cfg = _custom(synth.ModelShape(2, 256, heads, kv, 512, 1008, head_dim=dh), 1)
    cfg.n_prompt = 864          # room for 1024 positions, the most that one launch takes
    amd, ctx, tm, _ = _setup(cfg, gamma_max=15)
    ids = synth.prompt_tokens(1000, 1008, 7).tolist()
    for context in (0, 1, 33, 64, 447, 479, 480, 481, 512, 899):
        ctx.prefill(ids[:context + 1])
        ocm = transformer.CachedModel(tm, 1024)
        if context:
            ocm.feed(ids[:context])
        ref = ocm.feed(ids[context:context + 16])
        for m in (1, 2, 4, 5, 8, 9, 16):
            got = ctx.verify(ids[context:context + m], want_logits=True)
            assert _rel_err(got, ref[:m]) <= LOGIT_TOL, (context, m)
            ctx.rollback_kv(amd.SPEC_TARGET, context)
        # what a window left in the cache (over a page boundary at 64), read back by the next one
        ctx.verify(ids[context:context + 4])
        got = ctx.verify(ids[context + 4:context + 7], want_logits=True)
        assert _rel_err(got, ref[4:7]) <= LOGIT_TOL, context
        print(f"  heads {heads}/{kv} x {dh}, context {context}: ok", flush=True)
    ctx.close()
