"""Decode attention at the edges of its chunks, pages, row tiles and kernels (run with -m gpu)."""
import numpy as np
import pytest

import synth
from oracle import transformer
from tests.test_gpu_forward import LOGIT_TOL, _custom, _rel_err, _setup
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# heads, KV heads, head_dim; contexts around a chunk (32), a page (64), a round of the one-launch kernel (7 chunks); new
# tokens around a row tile (16) and over a page boundary.  A context of room for more than 1216 tokens takes the split
# kernel, whatever it holds.
@pytest.mark.parametrize("heads,kv,dh", [(4, 4, 128), (8, 2, 64), (8, 1, 128)])
@pytest.mark.parametrize("room", [0, 1100])
def test_contexts_and_windows_around_every_boundary(heads, kv, dh, room):
    cfg = _custom(synth.ModelShape(2, 256, heads, kv, 512, 1008, head_dim=dh), 1)
    cfg.n_prompt = 400
    amd, ctx, tm, _ = _setup(cfg, gamma_max=31, extra_seq=room)
    ids = synth.prompt_tokens(600, 1008, 7).tolist()
    for context in (0, 1, 31, 32, 33, 63, 64, 65, 223, 225, 256, 383):
        ctx.prefill(ids[:context + 1])
        ocm = transformer.CachedModel(tm, 512)
        if context:
            ocm.feed(ids[:context])
        ref = ocm.feed(ids[context:context + 32])
        for m in (1, 4, 5, 16, 17, 32):
            got = ctx.verify(ids[context:context + m], want_logits=True)
            err = _rel_err(got, ref[:m])
            assert err <= LOGIT_TOL, (context, m, err)
            ctx.rollback_kv(amd.SPEC_TARGET, context)
        # what a window left in the cache, read back by the next one
        ctx.verify(ids[context:context + 17])
        got = ctx.verify(ids[context + 17:context + 20], want_logits=True)
        assert _rel_err(got, ref[17:20]) <= LOGIT_TOL, context
        print(f"  heads {heads}/{kv} x {dh}, room {room}, context {context}: ok", flush=True)
    ctx.close()
