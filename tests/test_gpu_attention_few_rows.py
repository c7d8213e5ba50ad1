"""Decode attention of few query rows over a context of up to 1216 positions (run with -m gpu)."""
import pytest

import synth
from oracle import transformer
from tests.test_gpu_forward import LOGIT_TOL, _custom, _rel_err, _setup
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# contexts around a chunk, a page, the chunks that a workgroup has in flight at once (7 waves, two each: 448 positions) and
# the next round of them, and the last positions there is room for; 512 positions of room, 1024, and 1216, the most that one launch takes
@pytest.mark.parametrize("heads,kv,dh", [(2, 2, 128), (4, 2, 64), (8, 1, 128)])
@pytest.mark.parametrize("room", [512, 1024, 1216])
def test_contexts_around_the_rounds_of_chunks(heads, kv, dh, room):
    cfg = _custom(synth.ModelShape(2, 256, heads, kv, 512, 1008, head_dim=dh), 1)
    cfg.n_prompt = room - 160          # with 64 tokens to generate, the ring of drafts and a page to spare
    amd, ctx, tm, _ = _setup(cfg, gamma_max=15)
    max_seq = room - 64
    ids = synth.prompt_tokens(1200, 1008, 7).tolist()
    for context in (0, 1, 33, 64, 224, 225, 432, 447, 448, 449, 479, 480, 481, 512, 672, 673, 896, 899, 1120, max_seq - 16):
        if context + 16 > max_seq:
            continue
        ctx.prefill(ids[:context + 1])
        ocm = transformer.CachedModel(tm, room)
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
