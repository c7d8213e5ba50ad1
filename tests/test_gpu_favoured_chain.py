"""Which chain's waves issue first changes no bit of what either model computes (run with -m gpu)."""
import numpy as np
import pytest

import synth
from tests.test_gpu_stale_cache import model
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# 8 target layers and a draft of the first: one draft pass is 0.2 target passes, so windows of 1 put the target in front, of 5
# neither and of 16 the draft.  Rows of every projection layout: up to 8 tokens, one row tile and two, K slices.
@pytest.mark.parametrize("shape", [(256, 4, 512), (2048, 16, 704)])
def test_the_favoured_chain_changes_no_bits(shape):
    import paper_2408_11850_amd as amd
    d, heads, ffn = shape
    target = model(synth.ModelShape(8, d, heads, heads, ffn, 1008), 3)
    draft = target.prefix(1, synth.ModelShape(1, d, heads, heads, ffn, 1008))
    ids = synth.prompt_tokens(90, 1008, 7).tolist()
    seen = []
    for gamma in (1, 5, 16):
        ctx = amd.SpecContext(target, draft, gamma_max=gamma, max_seq=256, temperature=0.7)
        ctx.prefill(ids[:40])
        out = []
        for m in (1, 5, 12, 20, 32):
            out.append(ctx.verify(ids[40:40 + m], want_logits=True).copy())
            ctx.rollback_kv(amd.SPEC_TARGET, 39)
        out.append([ctx.draft_step(0.37, want_token=True) for _ in range(2)])
        seen.append(out)
        ctx.close()
    for other in seen[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(seen[0], other))
